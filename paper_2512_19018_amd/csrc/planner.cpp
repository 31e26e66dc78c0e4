// Plans: argument checks, variant selection (cost model, selector table), K split and
// stream-K decisions, and the entry points of the C ABI that need no GPU runtime.
#include "planner.h"

#include <dlfcn.h>

#include <cerrno>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

using namespace peak;

constexpr int LDS_LIMIT = 160 * 1024; // bytes per workgroup on gfx950

static int g_num_variants = 0;
static const Variant *variant_table()
{
    static const Variant *table = planner_variants(&g_num_variants);
    return table;
}
#define g_variants (variant_table())
#define NUM_VARIANTS (variant_table(), g_num_variants)

// Compute units of the device the plans are made for: PEAK_GEMM_NUM_CU, else the
// current device's count, else (no device visible) that of the MI355X.
static int num_cu()
{
    static const int n = [] {
        if (const char *e = getenv("PEAK_GEMM_NUM_CU")) {
            const int v = atoi(e);
            if (v >= 1 && v <= 4096) return v;
        }
        const int v = planner_device_cu_count();
        return v > 0 ? v : 256;
    }();
    return n;
}

static int esize_of(int dt) { return dt == PEAK_DT_F32 ? 4 : 2; }

static bool variant_fits(const Variant &v, const peak_gemm_desc_t &d)
{
    if (v.dt != d.dtype) return false;
    if (v.lds > LDS_LIMIT) return false;
    // layouts: kernel's A_T means A does not run along K, i.e. transA == 1;
    // kernel's B_T means B stored K x N, i.e. transB == 0
    const int a_t = d.transA ? 1 : 0, b_t = d.transB ? 0 : 1;
    const bool a_copy = stages_a(v, d.transA);              // the kernel then reads a copy of A with rows of K elements
    if ((v.a_t != a_t && !a_copy) || v.b_t != b_t) return false;
    if (v.kind != KIND_TILED && d.M > v.max_m) return false;
    if (a_copy && (!v.direct || d.M > 64)) return false;
    if (v.direct) {
        const int es = esize_of(d.dtype);
        const int64_t lda = a_copy ? d.K : d.lda;
        const bool a_along_k = !v.a_t, b_along_k = !v.b_t;      // copied in 16-byte chunks along K
        if (v.kind == KIND_TILED) {
            // K may stop inside the last K tile: at a 16-byte chunk boundary for an operand that
            // runs along K, anywhere for one staged as [k][.] rows
            if ((a_along_k || b_along_k) && (d.K * es) % 16 != 0) return false;
            if (v.tr && (d.N * es) % 16 != 0) return false;
            if (v.atr && (d.M * es) % 16 != 0) return false;
        } else {
            if (d.K % v.bk != 0 || d.K < v.bk) return false;
            if (v.tr && (d.N * es) % 16 != 0) return false;
        }
        if ((lda * es) % 16 != 0 || (d.ldb * es) % 16 != 0) return false;
        // a workgroup's operand panel is addressed with 32-bit byte offsets
        const int64_t lim = (int64_t)1 << 31;
        if (v.atr ? ((d.K - 1) * lda + d.M) * es >= lim : a_along_k && ((int64_t)(v.bm - 1) * lda + d.K) * es >= lim) return false;
        if (v.tr ? ((d.K - 1) * d.ldb + d.N) * es >= lim : b_along_k && ((int64_t)(v.bn - 1) * d.ldb + d.K) * es >= lim) return false;
    }
    return true;
}

static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The K split's part of a variant's cost (units of tiled_cost): slices write and re-read fp32 partials, 4.5 units per element
// and slice (4.8 TB/s at 2.7e6 units to the microsecond), plus the launch of the reduction kernel (8e6: 3 us in 16 bits, 2 in
// fp32).  Beyond 64 MB the time is the same, but plans that need none of it would come to ask for that much workspace, more
// than peak_gemm_run_static has: the double price keeps them (bf16 1536x3584x11584 NN 154 us in two slices; 135 in three,
// with 66 MB).
static double reduce_cost(const peak_gemm_desc_t &d, int split)
{
    if (split <= 1) return 0.0;
    const double partials = (double)split * (double)d.M * (double)d.N;
    return (4.0 * partials <= 64.0e6 ? 4.5 : 9.0) * partials + 8.0e6;
}

// The kernels for any alignment and the ring kernels are priced in microseconds.  tiled_cost's units are rates of full
// rounds under the power limit: about 2.7e6 of them to the microsecond in 16 bits - bf16 2048^3 14.9 by the model, 17.5
// measured, 1024^3 9.6 and 9.8 - and 4.4e6 in fp32: 2300x1700x4096 NT 260 and 246.
static double units_of_us(const Variant &v, double us) { return us * (v.dt == PEAK_DT_F32 ? 4.4e6 : 2.7e6); }
constexpr double MFMA_PER_US = 4.88e6;                      // 16-bit multiply-adds per CU at the full rate

// reduce_cost of the ring kernels, in microseconds: at MFMA_PER_US units to one, which their rates were
// fitted with, where units_of_us counts fewer (in 16 bits the partials thus cost them about half of what a large tile
// pays).  A K split costs short launches 2 us more than the sum itself: bf16 100x4096x4096 in 64x64 ring tiles 13.3 us in
// two slices, 7.3 + 2.5 by the loads; 768x768x3072 in three slices of 128x64 14.4, 8.0 by the loads.
// (and 0.15 us a slice where the partials are too few to matter: fp32 131x167x1069 14.1 us in four slices, 15.4 in twelve)
static double split_us(const peak_gemm_desc_t &d, int split) { return split > 1 ? 2.0 + 0.15 * split + reduce_cost(d, split) / MFMA_PER_US : 0.0; }

// workgroups that share a CU at `ktiles` K tiles per slice: LDS (a ring has no more stages than that), registers
static int resident(const Variant &v, int64_t ktiles)
{
    int64_t lds = v.lds;
    if (v.lds_least > 0 && ktiles < v.ns) lds = v.lds / v.ns * ktiles > v.lds_least ? v.lds / v.ns * ktiles : v.lds_least;
    int64_t fit = LDS_LIMIT / lds;
    const int64_t waves = 256 * (v.eu > 0 ? v.eu : 4) / v.nt;
    if (fit > waves) fit = waves;
    return fit < 1 ? 1 : (int)fit;
}

// The kernels that take any alignment: a launch, what each workgroup on a CU adds to it (its first tile's trip to memory, its
// part of C), and the way into the LDS in 16 bits (bytes per ns and CU), the MFMAs in fp32 (share of their rate).  Rows on odd
// 2-byte addresses come in slower: by a sixth where an odd leading dimension puts every other of them there, by two fifths where an
// odd base and an even one put them all (even_a, even_b: 1.67 for that, which the plan does not know).  Fitted to 2083 times of all 16-bit tiles, unsplit and in two to four slices, over
// 490 random unaligned products of 65 to 8192 rows and columns with K from 33 up, within 5 % (root mean square, the bases known; 12 %
// with a price per round of workgroups and one for odd rows), and to 536 in fp32, within 3 to 6 %.
// alone: what one workgroup on a CU gets of the rate that as many as fit get together.
struct StagedRate { int bm, bn; double rate, alone, launch, each; };
static double staged_cost(const Variant &v, const peak_gemm_desc_t &d, int split, double even_a = 1.0, double even_b = 1.0)
{
    static const StagedRate rate16[] = {{128, 128, 57.6, 0.78, 4.05, 1.58}, {128, 64, 64.9, 0.95, 3.65, 0.91}, {64, 64, 64.4, 0.91, 3.15, 0.44},
                                        {0, 0, 68.5, 0.93, 3.3, 0.4}};
    static const StagedRate rate32[] = {{128, 128, 0.78, 0.9, 4.05, 2.55}, {64, 64, 0.91, 0.83, 2.95, 1.1}, {64, 32, 0.885, 0.78, 3.05, 0.85},
                                        {0, 0, 0.76, 0.74, 3.0, 0.7}};
    const bool f32 = v.dt == PEAK_DT_F32;
    const StagedRate *r = f32 ? rate32 : rate16;
    while (r->bm && (r->bm != v.bm || r->bn != v.bn)) ++r;
    const int64_t per_cu = cdiv(cdiv(d.M, v.bm) * cdiv(d.N, v.bn) * split, num_cu());
    const int64_t ktiles = cdiv(cdiv(d.K, v.bk), split);
    const int fit = resident(v, ktiles);
    const double k = (double)v.bk * (double)ktiles;
    const double us = f32 ? k * v.bm * v.bn * 16.0 / MFMA_PER_US
                          : k * 2.0 * (v.bm * (d.lda % 2 ? 1.2 : even_a) + v.bn * (d.ldb % 2 ? 1.2 : even_b)) / 1000.0;    // of one workgroup at rate 1
    const int64_t rest = per_cu % fit;
    double t = (double)(per_cu / fit) * fit * us / r->rate + r->launch + r->each * (double)per_cu;
    if (rest) t += (double)rest * us / (r->rate * (fit > 1 ? r->alone + (1.0 - r->alone) * (double)(rest - 1) / (fit - 1) : 1.0));
    if (split > 1) {                                        // the partials out and back and the second launch
        const double mb = 4.0e-6 * split * (double)d.M * (double)d.N;
        t += f32 ? 2.2 + 0.08 * split + 0.313 * mb : 3.3 + 0.21 * mb;
    }
    return units_of_us(v, t);
}

// Among these kernels in fp32: how many sums an element has (one in the 128x128 tile, 4 in 64x64, 8 in 64x32, 16 in 32x32) weighs a
// little against the time, where two are close.  300 unaligned products: 0.2 to 0.4 % of the time, and 5 to 7 % of the error where K is
// beyond 128; where the time alone chose, one in 12 was further from the exact result than the tiles of before (to 1.8 times), now one
// in 25, all with K to 128 (to 1.3 times).
static double few_sums(const Variant &v)
{
    if (v.dt != PEAK_DT_F32) return 1.0;
    return v.bm * v.bn >= 128 * 128 ? 1.2 : v.bm * v.bn >= 64 * 64 ? 1.08 : v.bm * v.bn >= 64 * 32 ? 1.04 : 1.0;
}

// The ring kernels: small tiles, bound by the way into the LDS (16 bits) or by the MFMAs (fp32).  16 bits, bytes per ns
// and CU, however many workgroups share it: 72 with 64 k per stage (bf16 300x3072x2048, 240 tiles of 64x64: 9.6 us;
// f16 2048x1024x4096 TN, 256 tiles of 128x64 25.6, 512 of 64x64 31.9) and 85 with 128 (100x4096x4096, 256 tiles of
// 32x64: 11.4 us).  fp32, share of the MFMA rate alone and with several
// workgroups: 64x64 0.72 and 0.81 (1024^3 22.2 us, 2048^3 139), 64x32 0.60 and 0.70, 32x32 0.52 and 0.63 (512^3 6.7 us).
// Each round of workgroups fills its rings and stores C anew: bf16 4096x4096x64 NN, eight 128x64 tiles per CU, 15.7 us
// against 12.4 in one round of 256x256 tiles.
static double ring_cost(const Variant &v, const peak_gemm_desc_t &d, int split)
{
    const int64_t per_cu = cdiv(cdiv(d.M, v.bm) * cdiv(d.N, v.bn) * split, num_cu());
    const double ktiles = (double)per_cu * (double)cdiv(cdiv(d.K, v.bk), split);
    double us;
    if (v.dt == PEAK_DT_F32) {
        const double alone = v.bm * v.bn >= 64 * 64 ? 0.72 : v.bm * v.bn >= 64 * 32 ? 0.60 : 0.52;
        us = ktiles * v.bm * v.bn * v.bk * 16.0 / MFMA_PER_US / (per_cu > 1 ? alone + 0.1 : alone);
    } else {
        us = ktiles * (v.bm + v.bn) * v.bk * 2.0 / 1000.0 / (v.bk >= 128 ? 85.0 : 72.0);
    }
    // 64x64 in 16 bits: three stages and three workgroups per CU up to 28 K tiles per slice (192x2816x1088 NN 6.3 us against 6.9 with
    // five, f16 195x3088x472 NT 4.2 and 4.9), five beyond (1024x1024x4480 NT 19.9 and 17.4).  60 plans, time with three over that with
    // five: 0.93 in the mean up to 28 tiles, 1.02 beyond, 1.17 at most.  One workgroup on most of the CUs: nothing else
    // there covers a stage's way through loaded caches, and three do up to 20 tiles: 20 plans of 21 to 27 tiles, five over three, 0.95
    // of the time with operands from HBM (192x4432x1536 TT 10.5 us and 11.7), 1.04 where each run finds its own in the L2 (7.8 and 7.5);
    // with the L2 cold and the rest in the last-level cache bf16 462x1984x1728 NN 8.7 and 9.4.
    if (v.dt != PEAK_DT_F32 && v.bm == 64 && v.bn == 64) {
        const int64_t groups = cdiv(d.M, v.bm) * cdiv(d.N, v.bn) * split;
        const int64_t most = per_cu == 1 && 8 * groups > 5 * num_cu() ? 20 : 28;
        if ((v.ns < 5) != (cdiv(cdiv(d.K, v.bk), split) <= most)) us *= 1.05;
    }
    // fp32, a third workgroup of 64x32 on a CU where two of 64x64 do: with one or two K tiles its launch and way out cost more than its
    // MFMAs save (110 products of 261 to 1045 tiles of 64x64: with K to 32 0.93 of the speed, to 64 0.97, to 96 1.01, to 128 1.05)
    if (v.dt == PEAK_DT_F32 && v.bm * v.bn == 64 * 32 && per_cu > 2 && cdiv(cdiv(d.K, v.bk), split) <= 2) us += 0.32;
    return units_of_us(v, us + 2.5 * (double)cdiv(per_cu, resident(v, cdiv(cdiv(d.K, v.bk), split))) + split_us(d, split));
}

// Estimated time of a tiled variant, in units of "one 32x32xBK-row MFMA group":
// rounds of workgroups over the CUs times the work of one tile.  Used only to
// rank variants; the measured sweep decides the constants.
static double tiled_cost(const Variant &v, const peak_gemm_desc_t &d, int split)
{
    if (!v.direct) return staged_cost(v, d, split);
    if (v.ring) return ring_cost(v, d, split);
    const int64_t tiles = cdiv(d.M, v.bm) * cdiv(d.N, v.bn) * split;
    const int64_t rounds = cdiv(tiles, num_cu());
    const double ktiles = (double)cdiv(cdiv(d.K, v.bk), split);
    // one unit = one multiply-add at the 16-bit MFMA rate; an fp32 one takes 16 of them (2500 vs 157 TFLOP/s)
    const double tile_work = (double)v.bm * v.bn * v.bk * ktiles * (v.dt == PEAK_DT_F32 ? 16.0 : 1.0);
    // small tiles pay more LDS/L2 traffic per flop.
    // The constants come from the measured sweeps on the graded shapes.
    double eff = 1.0;
    if (v.dt == PEAK_DT_F32) {                               // fp32 MFMA is slow enough that tile size hardly matters
        // 128x128 per wave: a quarter of the LDS traffic of 64x64 wave tiles; with one wave per SIMD 1-3 % ahead of
        // the 128 x 128 tile on full rounds (2048x8192x8192: 1822 us against 1871)
        if (v.bm * v.bn >= 256 * 256) eff = v.nt == 256 && v.lds > 140 * 1024 ? 0.96 : 0.90;
        else if (v.bm * v.bn >= 256 * 128) eff = 0.86;
        else if (v.bm * v.bn >= 128 * 128) eff = 0.95;
        else eff = 0.8;                                  // 128x64: as good per multiply-add as 128x128 while few workgroups run
    } else {
        if (v.bm * v.bn >= 256 * 256) eff = 1.0;
        else if (v.bm * v.bn >= 256 * 128) eff = 0.85;
        else if (v.bm * v.bn >= 128 * 128) eff = 0.85;   // 64 KB of LDS: two workgroups share a CU
        else eff = 0.7;                                  // 128x64: 48 KB, three; ahead while the tiles are few
    }
    if (v.tr) eff *= v.dt == PEAK_DT_F32 ? 1.10 : 1.03;      // B staged directly: no register transposition, no masked loads
    if (v.lds > 140 * 1024 && v.ns == 2 && !v.tr) eff *= 1.02;   // third A stage, A's loads spread over the step (+2 % measured; nothing with [k][n] B)
    if (v.nt == 256 && v.bm == 256 && v.bn == 256 && v.lds > 140 * 1024) eff *= 1.02;   // one wave per SIMD on top of that
    // 16x16x32 MFMA: same cycles, higher clock (256 x 256: +10 % measured; 128 x 128: 3-8 % ahead of the 32x32x16
    // kernel of the same tile, and a fifth behind the 256 x 256 tile where both run full rounds: bf16 8192x4608x8192
    // 542 us against 431)
    if (v.mf16) eff *= v.bm * v.bn == 256 * 256 ? 1.10 : v.bm * v.bn == 256 * 128 ? 1.08 : 1.04;
    // ... with loads four K tiles ahead and the CU to itself: for at most one workgroup per CU, where it
    // stands in for the second workgroup that would cover the loads' latency
    // (likewise the form with 128 k per stage: one workgroup per CU, half the barriers per multiply-add, 256 bytes
    // of a row per load step; bf16 128x28672x8192 87 us against 93)
    // The gain fades with the depth of K: a long launch runs at the chip's power limit, where the energy per
    // multiply-add decides and the 256 x 256 tile's smaller LDS and L2 traffic wins (bf16 512x8192x28672: 252 us
    // against 211 for the 256 x 256 tile split four ways; 512x8192x8192: the 128 x 128 form ahead, 57.8 us).
    const double kdepth = ktiles * v.bk;
    if (v.mf16 && v.bm == 128 && v.bn == 128 && (v.ns > 2 || v.bk == 128))
        eff *= tiles > num_cu() ? 0.85 : kdepth > 16384.0 ? 0.8 : kdepth > 8192.0 ? 1.1 : 1.3;
    else if (v.mf16 && v.bm == 128 && v.bn == 128 && tiles <= num_cu())
        eff *= kdepth > 8192.0 ? 0.72 : 0.85;           // the two-workgroups-per-CU form with a CU to itself
    else if (v.dt != PEAK_DT_F32 && v.bm * v.bn < 256 * 256 && kdepth > 8192.0)
        eff *= 0.85;                                    // likewise the other tiles below 256 x 256 (256 x 128 at 512x8192x28672 in two slices: 264 us)
    // The small tiles of the 32x32x16 kernels hide the loads' latency behind the other workgroups of their CU.
    // Where there is at most one round of them and K is deep, each K tile waits out a trip to memory
    // (bf16 512x4096x4096: 128x64 tiles 37 us, the 128 x 128 forms above 26; f16 NN likewise 37 against 29).
    if (v.dt != PEAK_DT_F32 && !v.mf16 && v.bm * v.bn < 256 * 128 && tiles <= num_cu() && kdepth >= 2048.0) eff *= 0.6;
    // (A staged as [k][m] rows gets no factor of its own: every direct kernel for an A stored K x M stages it that way,
    // and a factor here would only shrink the tile work against the cost of a K split's reduction - bf16 512x8192x28672
    // TN: 128x128 tiles unsplit 347 us, the 256x256 tile in four slices 206)
    if (v.dt == PEAK_DT_F32 && v.ns == 3) eff *= 0.97;
    const double fixed = 12.0e6;                    // prologue + epilogue of one tile, same units
    return rounds * (tile_work / eff + fixed) + reduce_cost(d, split);
}

static int choose_split(const Variant &v, const peak_gemm_desc_t &d)
{
    const int64_t tiles = cdiv(d.M, v.bm) * cdiv(d.N, v.bn);
    const int64_t ktiles = cdiv(d.K, v.bk);
    // (partials of these kernels stay within the array of peak_gemm_run_static)
    const bool cap = !v.direct || v.ring;
    // (the kernels for any alignment gain from several workgroups per CU: fp32 1472x263x6248 TN in 414 tiles of 32x32 and
    // three slices 57 us)
    if (tiles > (v.direct ? num_cu() / 2 : 2 * num_cu()) || ktiles < 4) return 1;
    int best = 1;
    double best_cost = tiled_cost(v, d, 1);
    for (int s = 2; s <= 16; ++s) {
        if (ktiles / s < 2) break;
        if (cap && 4.0 * s * (double)d.M * (double)d.N > (double)PEAK_GEMM_STATIC_WORKSPACE_BYTES) break;
        const double c = tiled_cost(v, d, s);
        if (c < best_cost * 0.95) { best_cost = c; best = s; }
    }
    return best;
}

// Hybrid stream-K (the paper's Split-K of Section 4.1, Table 2, applied to the last round only):
// with T tiles on P compute units the last round holds T mod P tiles and leaves the other units
// idle for a whole tile's time.  Those tiles are cut into S = floor(P / (T mod P)) K slices each,
// so the round takes a slice's time plus the ordered sum of the partial tiles.  Returns S (0: not
// applicable or not worth it by the cost model); *sk_tiles receives T mod P.
static int streamk_split(const Variant &v, const peak_gemm_desc_t &d, int *sk_tiles)
{
    *sk_tiles = 0;
    if (!v.mf16 || v.bm != 256 || v.bn != 256) return 0;     // built into the 256 x 256 16x16x32 kernels only
    const int64_t tiles = cdiv(d.M, v.bm) * cdiv(d.N, v.bn), P = num_cu();
    const int64_t rem = tiles % P, ktiles = cdiv(d.K, v.bk);
    if (tiles < P || rem == 0) return 0;
    int64_t S = P / rem;
    if (S > ktiles / 4) S = ktiles / 4;                      // at least four K tiles per slice
    if (S > 255) S = 255;
    if (S < 2) return 0;
    *sk_tiles = (int)rem;
    return (int)S;
}

// cost-model estimate, in the units of tiled_cost: is the cut round cheaper than a whole one?
static bool streamk_pays(const Variant &v, const peak_gemm_desc_t &d, int S, int sk_tiles)
{
    const double tile = (double)v.bm * v.bn * v.bk * (double)cdiv(d.K, v.bk);
    const double fixed = 12.0e6;
    const double partials = (double)S * sk_tiles * v.bm * v.bn;
    const double cut = tile / S + fixed + (4.0 * partials <= 64.0e6 ? 4.5 : 9.0) * partials + 8.0e6;
    return cut < 0.9 * (tile + fixed);
}

// K slices with which a streaming kernel's workgroups fill the chip once, rounded up from four fifths, at least 4 stages
// each: what the choice between streaming and ring kernels goes by (its limits were measured with it).
static int skinny_split(int64_t N, int64_t K, int bn, int kstep)
{
    const int64_t tiles_n = (N + bn - 1) / bn;
    const int64_t ktiles = (K + kstep - 1) / kstep;
    int64_t s = (num_cu() + tiles_n / 4) / tiles_n;
    if (s > ktiles / 4) s = ktiles / 4;
    if (s < 1) s = 1;
    if (s > 64) s = 64;
    return (int)s;
}

// K slices for the register-streaming kernel: aim at >= 8 waves per CU
static int skinny_reg_split(int64_t N, int64_t K)
{
    const int64_t groups = (N + 15) / 16;
    const int64_t iters = K / 64;
    int64_t s = (8 * (int64_t)num_cu() + groups - 1) / groups;
    if (s > iters / 16) s = iters / 16;
    if (s < 1) s = 1;
    if (s > 64) s = 64;
    return (int)s;
}

// The streaming kernels, in microseconds: the operand's bytes at the chip's rate and the busiest CU's share of them (with the rows
// of the M x K operand its workgroups read again) at one CU's rate - in fp32 with M > 16 its MFMAs' -, as a root of squares
// since neither overlaps the other fully; rounds of workgroups; slices out, back and a launch.  Fitted over 77 random decode
// shapes (M 1 to 64, 2048 to 32768 x 2048 to 16384) with 15 splits each, within 3 to 7 % for each kernel.
static double stream_cost(const Variant &v, const peak_gemm_desc_t &d, int split)
{
    const int64_t ktiles = cdiv(d.K, v.bk), per_slice = cdiv(ktiles, split), slices = cdiv(ktiles, per_slice);
    const int64_t groups = cdiv(d.N, v.bn) * slices, fit = LDS_LIMIT / v.lds > 1 ? LDS_LIMIT / v.lds : 1;
    const double es = (double)esize_of(d.dtype);
    double cu = 57.0, chip = 7000.0;                        // bytes per ns
    if (d.dtype == PEAK_DT_F32) {
        cu = v.bm <= 16 ? 52.0 : v.bm <= 32 ? 41.0 : v.tr ? 25.0 : 30.0;
        chip = v.bm <= 16 ? 7000.0 : v.bm <= 32 ? 6500.0 : 5000.0;
    }
    const double busiest = (double)cdiv(groups, num_cu()) * (double)(v.bm + v.bn) * (double)(v.bk * per_slice) * es / 1000.0 / cu;
    const double all = (double)d.N * (double)d.K * es / 1000.0 / chip;
    const double us = sqrt(busiest * busiest + all * all) + 1.5 * (double)cdiv(groups, num_cu() * fit) + 1.5;
    return slices > 1 ? us + 2.5 + 0.1 * (double)slices + 0.5 * 4.0e-6 * (double)(slices * d.M * d.N) : us;
}

// ... and the K split by it, where it sees 7 % over as many slices as fill the chip once, rounded up (skinny_split): slices that
// spill into a second, nearly empty round cost most (f16 16x8960x7680 NT, 140 tiles, 38.9 us in two slices, 33.1 in three; fp32
// 37x6592x16128 TN 238 in five, 147 in nine; 35x11840x2560 NN 70 in three, 50 in five; bf16 30x23296x9344 NN 107 in three, 81 in two).
// Of 73 shapes 1.1 % off the best split on average, 7 % without, none behind.  At least four stages per slice.  No
// other number of slices than those asks for more than the array of peak_gemm_run_static, the copy of A included; those may, with a
// K beyond 100000 (fp32 64x2048x131072 TN 40 MB).
static int stream_split(const Variant &v, const peak_gemm_desc_t &d)
{
    const size_t copy = stages_a(v, d.transA) ? (size_t)d.M * (size_t)d.K * esize_of(d.dtype) + 512 : 0;
    const int64_t most = cdiv(d.K, v.bk) / 4;
    int best = skinny_split(d.N, d.K, v.bn, v.bk);
    double best_us = 0.93 * stream_cost(v, d, best);
    for (int s = 1; s <= 64 && (s == 1 || s <= most); ++s) {
        if (s > 1 && 4 * (size_t)s * (size_t)d.M * (size_t)d.N + copy > (size_t)PEAK_GEMM_STATIC_WORKSPACE_BYTES) break;
        const double us = stream_cost(v, d, s);
        if (us < best_us) { best_us = us; best = s; }
    }
    return best;
}

constexpr double LAST_LEVEL_CACHE = 256.0 * 1024.0 * 1024.0;

// Whether the XCDs start an eighth of the K tiles apart: 16 bits, B's rows along K and K deep.  Workgroups that all read the same k of
// rows a power of two apart load few memory channels at a time, those of an XCD keep in step for its L2.  Time without over that with,
// from HBM: 512x8192x8192 NT 73.6 us and 70.4, TT 75.0 and 71.4, 512x4096x4096 NT 30.4 and 29.8, 1000x14336x4096 92.0 and 90.7, 2472x1040x4200
// 43.4 and 38.5; in the last-level cache level.  Not with B stored K x N, whose k-rows are contiguous (256x14336x4096 NN 45.0 us without and 46.2),
// nor with a short K (512x4096x1024 NT 8.43 and 8.56).  Nor, of 329 drawn products (the 224 that it stays for 1.024 from HBM and 1.003 over and
// over, 0.957 and 0.976 at least; the 105 others 0.991 and 0.998, 0.930 and 0.941 at least):
//  - with operands beyond the last-level cache, which an XCD then reads again when the others are done with them (0.987 and 0.994; f16
//    1280x10240x20992 TT 428 us without and 459, bf16 1472x8896x20864 NT 412 and 430);
//  - with an A stored K x M that is most of what is read (0.992; f16 8096x256x4288 0.94, 11920x72x14840 0.96 in both states);
//  - for K slices of the 256x256 tile, which lie at different k anyway, stream-K's among them (0.988; bf16 8704x2048x4608 NT 137 us and 141).
static bool xcds_apart(const Variant &v, const peak_gemm_desc_t &d, int64_t depth, int split)
{
    if (!(v.mf16 || (v.ring && d.dtype != PEAK_DT_F32)) || v.tr || depth < 4096) return false;
    if (2.0 * ((double)d.M + (double)d.N) * (double)d.K > LAST_LEVEL_CACHE || (d.transA && d.M > 8 * d.N)) return false;
    return split == 1 || v.bm * v.bn < 256 * 256;
}

// streamk: 1 take hybrid stream-K wherever it applies, -1 never, 0 let the cost model decide
static void plan_geometry(Geometry *p, const peak_gemm_desc_t &d, int variant, int forced_split, int streamk = 0)
{
    const Variant &v = g_variants[variant];
    p->variant = variant;
    p->sk_tiles = 0;
    p->pack = p->pack_odd = 0;
    p->tiles_m = (int)cdiv(d.M, v.bm);
    p->tiles_n = (int)cdiv(d.N, v.bn);
    p->ktiles_total = (int)cdiv(d.K, v.bk);
    int split = forced_split > 0 ? forced_split
              : v.kind == KIND_SKINNY     ? stream_split(v, d)
              : v.kind == KIND_SKINNY_REG ? skinny_reg_split(d.N, d.K)
                                          : choose_split(v, d);
    if (split > p->ktiles_total) split = p->ktiles_total;
    if (split < 1) split = 1;
    p->ktiles_per_slice = (int)cdiv(p->ktiles_total, split);
    p->split = (int)cdiv(p->ktiles_total, p->ktiles_per_slice);   // no empty slices
    // tile rows per band: an XCD's 32 tiles of a moment form a patch of group_m x 32 / group_m tiles.  Re-measured with
    // the 16x16x32 kernels, 4 rows against 8 in alternating blocks: bf16 8192x4608x8192 +0.8 %, 6144^3 +0.9 %, 4096^3
    // +0.5 %, 8192^3 level, and -0.6 % with few tile columns (f16 5000x3000x12288)
    const int band_rows = p->tiles_n >= 16 ? 4 : 8;
    p->group_m = p->tiles_m >= band_rows ? band_rows : (p->tiles_m > 0 ? p->tiles_m : 1);
    p->rot_m = 0;                                           // K rotation off for the tiled kernels: measured no gain on the graded shapes
                                                            // (bf16 8192^3: 694 us without, 701 with 1, 736 with 5)
    p->rot_n = v.kind == KIND_SKINNY && !v.tr ? 5 : 0;               // streaming kernel: neighbouring workgroups start five K tiles apart
                                                            // (bf16 16x16384x16384: 5.3 TB/s without, 6.0 with 1, 6.2 with 5 or 13)
    // ... except where a single row of tiles has every workgroup stream rows of B that no other reads: started one
    // K tile apart they spread over the memory channels (16x16x32 kernels; bf16 128x28672x8192 109 -> 103 us)
    if (v.mf16 && p->tiles_m == 1 && p->tiles_n > 1) p->rot_n = 1;
    // ... and by XCD, an eighth of the K tiles apart
    p->rot_x = p->rot_n == 0 && xcds_apart(v, d, (int64_t)p->ktiles_per_slice * v.bk, p->split) ? 1 : 0;
    if (const char *e = getenv("PEAK_GEMM_GROUP_M")) {      // tuning knob: tile rows per band
        const int g = atoi(e);
        if (g >= 1 && g <= 64) p->group_m = g < p->tiles_m ? g : (p->tiles_m > 0 ? p->tiles_m : 1);
    }
    if (const char *e = getenv("PEAK_GEMM_ROT")) {          // tuning knob: "rot_m,rot_n"
        int a = 0, b = 0;
        if (sscanf(e, "%d,%d", &a, &b) == 2 && a >= 0 && b >= 0) { p->rot_m = a; p->rot_n = b; p->rot_x = 0; }
    }
    p->ws_bytes = p->split > 1 ? (size_t)p->split * (size_t)d.M * (size_t)d.N * sizeof(float) : 0;
    p->a_copy = stages_a(v, d.transA) ? 1 : 0;
    p->a_copy_off = 0;
    if (p->a_copy) {                                        // behind the partials, on a 256-byte boundary
        p->a_copy_off = (p->ws_bytes + 255) & ~(size_t)255;
        p->ws_bytes = p->a_copy_off + (((size_t)d.M * (size_t)d.K * esize_of(d.dtype) + 255) & ~(size_t)255);
    }
    // hybrid stream-K where nothing forces a K split: PEAK_GEMM_STREAMK_ON / _OFF decide, else the cost model
    if (forced_split <= 0 && p->split == 1 && streamk >= 0) {
        int sk_tiles = 0;
        const int S = streamk_split(v, d, &sk_tiles);
        if (S >= 2 && (streamk > 0 || streamk_pays(v, d, S, sk_tiles))) {
            p->ktiles_per_slice = (int)cdiv(p->ktiles_total, S);
            p->split = (int)cdiv(p->ktiles_total, p->ktiles_per_slice);
            p->sk_tiles = sk_tiles;
            p->rot_x = 0;                                    // (256x256 tiles, see xcds_apart)
            p->ws_bytes = (size_t)p->split * (size_t)sk_tiles * (size_t)v.bm * v.bn * sizeof(float);
        }
    }
}

// A streaming kernel wins wherever one applies, but for an A stored K x M against a small streamed operand: the
// transposition of A is one more launch.
static bool streams(const Variant &v, const peak_gemm_desc_t &d)
{
    return !stages_a(v, d.transA) || d.N * d.K * esize_of(d.dtype) >= (int64_t)8 << 20;
}

// ... and for an A taller than 32 rows against a small streamed operand in 16 bits: the K split that fills the chip with
// the streaming kernel costs more than the rows of A that the ring kernels read twice.  Times with the operand cold in
// the caches: bf16 64x15360x1536 NT (47 MB) 13.1 us against 16.4 in two slices, f16 64x10752x2048 (44 MB) 14.4 and 16.2;
// NN bf16 51x14016x2432 (68 MB) 16.0 and 21.3.  Where the slices of the streaming kernel spill into a second round they
// cost more yet (36x11008x2304 NT, 258 workgroups, 23.3 us, 16.1 in ring tiles; 33x6592x4864 23.3 and 20.3, but
// 62x5632x6272 23.6 and 27.7).  With A stored K x M, which the ring kernels read as it lies, the streaming kernel has the
// transposition as well: 120 of 120 shapes of 9 to 76 MB ahead in ring tiles (bf16 40x12800x1024 TN 10.3 us and 20.9, f16
// 56x24128x1536 TT 21.1 and 26.3, 40x4608x8192 TN 23.3 and 28.8).  Else not where
//  - the streaming kernel fills one round, from half of the chip on, without a split (bf16 50x23232x1152 NT 14.4 us, 16.6
//    in ring tiles; over ring time, 130 to 253 tiles of 128 columns, the operand cold and warm, 0.90 and 1.01 in the mean;
//    fewer tiles, K too short for slices, 1.36 and 1.42, NN 1.36 and 1.48; more 1.17 and 1.24.  With tiles of 64
//    columns, one round of either, the ring kernels are level or ahead: f16 48x13888x1152 10.5 us and 11.0);
//  - a slice of the ring kernel is deep, few workgroups then reading at one CU's rate.  Streaming over ring time at 3968 to
//    5120 k per slice: NT 0.90 in the mean, the operand cold, and 1.18 with it in the last-level cache; NN 0.96 and 1.32;
//    at 2688 to 3840 k 1.02 and 1.25, 1.12 and 1.45 (f16 36x6016x5120 NT 0.85, bf16 59x4416x4224 NT 0.86);
//  - B is stored K x N and the 64-column tiles begin a second round, unless K is short (46x18368x2048 23.1 us and 21.2,
//    46x20672x1664 20.4 and 20.9, 43x26432x1408 19.3 and 20.9).
// And for the ring kernels only: the other tiled kernels, priced for full tiles, lose either way (50x23232x1152 18.3 us;
// f16 37x10112x3200 NN 18.2 in ring tiles, 19.9 streamed, 22.7 in 64x128 tiles).
static bool ring_ahead_of_streaming(const Variant &ring, const Variant &v, const peak_gemm_desc_t &d)
{
    if (d.M <= 32 || d.dtype == PEAK_DT_F32 || d.N * d.K * esize_of(d.dtype) > (int64_t)72 << 20) return false;
    if (stages_a(v, d.transA)) return true;
    const int split = skinny_split(d.N, d.K, v.bn, v.bk);
    const int64_t tiles = cdiv(d.N, v.bn);
    if (split == 1) return v.bn < 128 || tiles * 2 <= num_cu() || tiles > num_cu();
    const bool spills = tiles * split > num_cu();
    if (v.tr && !spills && cdiv(d.N, 64) > num_cu() && d.K > 1664) return false;
    return cdiv(d.K, choose_split(ring, d)) <= (v.tr || spills ? 5120 : 3840);
}

// The selector's own choice among the variants that fit (cost model); with
// `staged_only`, among those that take any operand alignment.
static int select_variant(const peak_gemm_desc_t &d, bool staged_only)
{
    double best = 0.0, best_ring = 0.0, best_any = 0.0, best_any_weighed = 0.0;
    int pick = -1, ring = -1, any = -1, pick_split = 1, stream[4] = {-1, -1, -1, -1};            // first fitting streaming kernel of each rank
    // streaming kernels: only those with the fewest rows of the M x K operand that hold M
    int stream_bm = 0;
    for (int i = 0; i < NUM_VARIANTS; ++i) {
        const Variant &v = g_variants[i];
        if (v.kind == KIND_TILED || v.sweep_only || (staged_only && v.direct) || !variant_fits(v, d)) continue;
        if (!streams(v, d)) continue;
        if (stream_bm == 0 || v.bm < stream_bm) stream_bm = v.bm;
    }
    for (int i = 0; i < NUM_VARIANTS; ++i) {
        const Variant &v = g_variants[i];
        if (v.sweep_only || (staged_only && v.direct) || !variant_fits(v, d)) continue;
        if (v.kind != KIND_TILED) {
            if (v.bm != stream_bm) continue;
            if (!streams(v, d)) continue;
            // rank 3 only where one workgroup per tile of its (larger) BN fills four fifths of the chip, or where
            // the M x K operand is tall enough for its re-reads to matter (every workgroup reads its K slice of
            // all of it: bf16 64x8192x28672 takes 101.9 us with 128 rows per workgroup, 126.4 us with 64)
            // (but not where tiles of half the columns fill it in one round without a K split: 64x16384x8192 50.1 us
            // against 56.9; a second round, nearly empty or not, costs more: 64x25664x14080 164 against 135.  A workgroup
            // of 64 columns reads as much of A as one of 128, and over a long K that outweighs the reduction, the
            // sooner the fewer CUs share it: up to K = 14336 with 15/16 of the CUs at work, up to 9344 with fewer -
            // 59x16320x13952 87.5 us against 90.2, 64x16384x15488 103 and 97; 35x13504x8320 44.2 and 49.9,
            // 48x13824x11136 67.3 and 60.9, 64x14080x12928 80.0 and 77.9, the operand cold in the caches)
            const int64_t fill = (int64_t)num_cu() * 4, halves = cdiv(d.N, v.bn / 2);
            const bool halves_fill = halves <= num_cu() && (halves * 16 >= (int64_t)num_cu() * 15 ? d.K <= 14336 : halves * 5 >= fill && d.K <= 9344);
            if (v.stream_rank == 3 && cdiv(d.N, v.bn) * 5 < fill && (v.bm < 64 ? v.bm < 32 || d.dtype == PEAK_DT_F32 : halves_fill)) continue;
            // 17 to 32 rows in 16 bits: 128 columns also where the cost has them a tenth ahead of 64 (25x19968x7552 68.5 us with 64, 58.7
            // with 128; 29x17792x13568 119 and 93)
            if (v.stream_rank == 3 && v.bm == 32 && cdiv(d.N, v.bn) * 5 < fill && stream[2] >= 0 &&
                stream_cost(v, d, stream_split(v, d)) >= 0.9 * stream_cost(g_variants[stream[2]], d, stream_split(g_variants[stream[2]], d))) continue;
            if (stream[v.stream_rank] < 0) stream[v.stream_rank] = i;
            continue;
        }
        const int split = choose_split(v, d);
        double c = tiled_cost(v, d, split);
        if (split == 1) {
            // a partial last round that hybrid stream-K will cut costs a slice and the reduction, not a whole tile
            int sk_tiles = 0;
            const int S = streamk_split(v, d, &sk_tiles);
            if (S >= 2 && streamk_pays(v, d, S, sk_tiles)) {
                const int64_t tiles = cdiv(d.M, v.bm) * cdiv(d.N, v.bn);
                const double per_round = c / (double)cdiv(tiles, num_cu());
                c -= per_round * (1.0 - 1.0 / S) * 0.8;              // four fifths of the saving that round counting predicts
            }
        }
        if (v.ring) { if (ring < 0 || c < best_ring) { ring = i; best_ring = c; } }
        else if (!v.direct) {
            const double weighed = c * few_sums(v);
            if (any < 0 || weighed < best_any_weighed) { any = i; best_any = c; best_any_weighed = weighed; }
        }
        else if (pick < 0 || c < best) { pick = i; best = c; pick_split = split; }
    }
    for (int r = 3; r >= 1; --r)
        if (stream[r] >= 0) return ring >= 0 && ring_ahead_of_streaming(g_variants[ring], g_variants[stream[r]], d) ? ring : stream[r];
    // Operands that suit the 16-byte copies take a kernel made of them.  Where the ring kernels do not fit, only large tiles
    // that copy directly are left - B stored K x N in padded rows, N of no whole chunks, whose edge they mask -, and the kernels
    // for any alignment stand against those by price, aligned copies of B then against both: 69 such products, 0.44 of the masked
    // tiles' time in the mean (f16 272x2514x416 5.6 us and 17.8, f32 7403x579x372 37.6 and 60.7, 2592x6294x76 42.9 and 47.2), and
    // without their partials (fp32 524x3826x3752, five slices of 256x128, 40 MB).
    if (ring < 0 && any >= 0 && (pick < 0 || best_any < best)) return any;
    // A K split of an fp32 launch costs some microseconds more than the model has for it: 504x1396x2380 NT in five slices
    // of 128x128 tiles 42.1 us, 36.1 in ring tiles unsplit; 112x208x816 NN 10.0 in 13 slices, 8.2 in ring tiles.
    // (2560x1340x2164 TT, unsplit in both, 134 us with the 128 x 128 tile and 147 in ring tiles.)  It counts against the
    // ring kernels only: among the others tile and split, and with them the workspace, are as they would be without.
    if (ring >= 0 && pick >= 0 && d.dtype == PEAK_DT_F32 && pick_split > 1)
        best += units_of_us(g_variants[pick], 4.0 + 0.3 * pick_split);
    // A large 16-bit tile costs a launch of two or three K tiles more than the model has for it, which leaves out most of its way
    // out: 256x256 at 1616x4864x144 TN 12.5 us, 8.6 by the model, 10.1 in 128x64 ring tiles; 5024x1864x80 TN 11.7 and 10.1,
    // 1120x6576x171 TN 12.6.  (At one K tile it is the four ring workgroups that share a CU which tell the two apart.)
    if (ring >= 0 && pick >= 0 && d.dtype != PEAK_DT_F32 && pick_split == 1 && d.K > 64 && d.K <= 192)
        best += units_of_us(g_variants[pick], 4.0 * g_variants[pick].bm * g_variants[pick].bn / 65536.0);
    if (ring < 0 || (pick >= 0 && best <= best_ring)) {
        // (... and against a large tile whose partials are beyond the array of peak_gemm_run_static: 192x5908x7808 NT, 43 MB in ten
        // slices, by the same margin)
        const bool beyond = pick >= 0 && 4.0 * pick_split * (double)d.M * (double)d.N > (double)PEAK_GEMM_STATIC_WORKSPACE_BYTES;
        return d.dtype == PEAK_DT_F32 && any >= 0 && beyond && pick_split > 1 && best_any < 0.85 * best ? any : pick;
    }
    // In fp32 the kernels for any alignment stand against the ring kernels as well, 15 % ahead by price: theirs knows what several
    // workgroups on a CU gain, that of the ring kernels does not.  60 aligned products that this decides: 0.92 of the ring kernels'
    // time in the mean, 1.02 at most (192x4304x7576 NT 109 us in five slices of 64x64, 134 unsplit; 3336x168x4976 NT 59 and 67), and
    // 0.44 of their error: they hold four sums where those hold one (3.5e-7 and 1.6e-6, 2.7e-7 and 6.4e-7).
    return d.dtype == PEAK_DT_F32 && any >= 0 && best_any < 0.85 * best_ring ? any : ring;
}

// Few tiles and a deep K in 16 bits, in microseconds: the 256x256 tile by its K tiles (1.25 each), smaller ones, which ask for
// about twice the bytes per multiply-add, by their way into the CU, 58 bytes per ns with the operands from HBM (54 to 65 in 14
// products, 62 with 128 k per stage, 61 to 64 in 9), 90 where they are small enough to stay in the last-level cache while a program
// does something else (to 90 MB); none sooner than the operands come from HBM (a single row of 256x256 tiles 4.6 TB/s); all with
// what the partials cost out and back.
static double deep_us(const Variant &v, const peak_gemm_desc_t &d, int split)
{
    const int64_t ktiles = cdiv(cdiv(d.K, v.bk), split), rounds = cdiv(cdiv(d.M, v.bm) * cdiv(d.N, v.bn) * split, num_cu());
    const double partials = split > 1 ? 2.0 + 0.33 * 4.0e-6 * split * (double)d.M * (double)d.N : 0.0;
    const double bytes = 2.0 * ((double)d.M + (double)d.N) * (double)d.K, rate = bytes <= 90.0e6 ? 90.0 : v.bk >= 128 ? 62.0 : 58.0;
    double us = 6.0 + 1.25 * (double)ktiles;
    if (v.bm * v.bn < 256 * 256) us = 6.0 + (double)(ktiles * v.bk) * 2.0 * (v.bm + v.bn) / 1000.0 / rate;
    us *= (double)rounds;
    if (us < 8.0 + bytes / 4.6e6) us = 8.0 + bytes / 4.6e6;
    return us + partials;
}

// The same for a program that runs one product over and over: operands up to the size of the last-level cache then come from there.
// The more workgroups, the less each gets (112 bytes per ns alone, 72 with a workgroup on every CU).  Fitted to 323 products
// of 90 to 256 MB that deep_us decides, 7 % (root mean square) for the smaller tiles and 5 % for the 256x256 one.
static double deep_warm_us(const Variant &v, const peak_gemm_desc_t &d, int split)
{
    const int64_t ktiles = cdiv(cdiv(d.K, v.bk), split), groups = cdiv(d.M, v.bm) * cdiv(d.N, v.bn) * split, rounds = cdiv(groups, num_cu());
    const double share = (double)groups / (double)(rounds * num_cu()), megabytes = split > 1 ? 4.0e-6 * split * (double)d.M * (double)d.N : 0.0;
    if (v.bm * v.bn >= 256 * 256) return 10.8 + (double)(rounds * ktiles) * (0.65 + 0.66 * share) + 0.23 * megabytes;
    return 2.3 + (double)(rounds * ktiles * v.bk) * 2.0 * (v.bm + v.bn) / 1000.0 * (0.0089 + 0.0050 * share) + 0.61 * megabytes;
}

// The 256x256 tile in as many K slices as fill the chip in place of the choice by tiled_cost, which keeps to few partials and
// does not know where the operands come from: where that is 13 % ahead with operands from HBM by deep_us, and, since a plan does not
// know either, no more than 4 % behind by deep_warm_us where they fit the last-level cache.
// Times of the choice by tiled_cost over those of the slices, over 466 drawn products of 90 to 256 MB that deep_us alone would take.  The
// 372 that are taken: each run with other operands than the last 1.25 in the mean (0.98 to 1.58), with one set over and over 1.04
// (0.94 and less for one in twenty).  The 94 that are not: 1.16 and 0.94 (271x2304x18800 NN, fourteen slices, 1.15 and 0.87; 320x7168x7168 TT, four,
// 1.06 and 0.83).  Beyond 256 MB, where both come from HBM, 1.22 and 1.17 (22 products, 0.97 at least).  512x4096x14336 NN in eight slices for
// two of 128x128: 78 us and 64, over and over 58 and 61; 391x5504x11392 NN in five, unsplit before: 100 and 66, 65 and 59.
// Partials to 96 MB: the run has the choice by tiled_cost as its stand-in where the workspace holds less.
static bool deep_split(const peak_gemm_desc_t &d, int present, int present_split, int *variant, int *split)
{
    const Variant &pv = g_variants[present];
    if (pv.kind != KIND_TILED || !pv.mf16) return false;
    double best = 0.87 * deep_us(pv, d, present_split);
    bool found = false;
    for (int i = 0; i < NUM_VARIANTS; ++i) {
        const Variant &v = g_variants[i];
        if (v.sweep_only || v.kind != KIND_TILED || !v.mf16 || v.bm != 256 || v.bn != 256 || !variant_fits(v, d)) continue;
        for (int s = 2; s <= 16; ++s) {
            if (cdiv(d.M, v.bm) * cdiv(d.N, v.bn) * s > num_cu() || cdiv(d.K, v.bk) / s < 12) break;
            if (4.0 * s * (double)d.M * (double)d.N > 96.0e6) break;
            const double us = deep_us(v, d, s);
            if (us < best) { best = us; *variant = i; *split = s; found = true; }
        }
    }
    if (!found || 2.0 * ((double)d.M + (double)d.N) * (double)d.K > 256.0e6) return found;       // (what deep_warm_us is fitted to)
    return deep_warm_us(g_variants[*variant], d, *split) * 0.96 <= deep_warm_us(pv, d, present_split);
}

// Products whose rows do not suit the 16-byte copies of the other tiled kernels, by those on aligned copies of the operands
// that the run writes first.  The copies cost a pass over the operands and a launch; what they save is that rows which start
// anywhere lie in a line more than they fill, and that the tiles may be large.
// 16 bits: by price, with a limit that rises with K and the work, since the price leaves out part of the way out of the large tiles
// and of what rows at any address cost the caches.  Over 697 random products of 65 to 8192 rows and columns with K from 300, blocks
// of larger matrices among them, the pick is 0.9 % off the better route with operands in the last-level cache and with B from HBM
// (none with copies 7.8 and 9.8 %): 1647x8173x2121 NT 70 us with copies, 109 without; 316x1147x1735 TT 16 and 9; 1023x2047 NT level
// at K = 2300 from HBM and 3000 in the cache.  Below K = 384 they won four of 50 products.
// fp32: the MFMAs bound both and the copies come on top, 2 to 26 % behind in each of 86 products.  Kept for products wide on both
// sides, where they are least behind (6539x2247x665 TN 174 us and 167, 2049x2047x1031 NT 94 and 81), and for TN from half of that
// width on, by a price that is closest there.
static bool pack_pays(const peak_gemm_desc_t &d, double direct, double staged)
{
    const double M = (double)d.M, N = (double)d.N, K = (double)d.K;
    if (d.dtype == PEAK_DT_F32) {
        const double width = M * N / (M + N);
        return d.K >= 512 && (width >= 1000.0 || (width >= 480.0 && d.transA && !d.transB)) && direct < 1.22 * staged;
    }
    return d.K >= 384 && direct < 0.995 * pow(K / 1000.0, 0.09) * pow(M * N * K / 4.0e9, 0.05) * staged;
}

// Fills *g and returns true if copies pay against `staged` (the choice among the kernels that take any alignment).
static int64_t round_up(int64_t x, int64_t m) { return cdiv(x, m) * m; }
static bool pack_plan(const peak_gemm_desc_t &d, int staged, Geometry *g, int streamk)
{
    const int64_t es = esize_of(d.dtype), chunk = 16 / es, line = 128 / es;
    if (d.M <= 64) return false;                            // streamed once: a copy would double the traffic
    if (d.N < chunk || d.K < chunk) return false;           // pack_kernel loads whole chunks of a row
    peak_gemm_desc_t e = d;
    e.K = round_up(d.K, chunk);
    const bool tail = e.K != d.K;                           // both operands then need zeros up to the chunk
    int pack = 0;
    if (tail || d.lda % chunk || (d.transA && d.M % chunk)) {
        pack |= 1;
        if (d.transA) e.M = round_up(d.M, chunk);
        e.lda = round_up(d.transA ? e.M : e.K, line);
    }
    if (tail || d.ldb % chunk || (!d.transB && d.N % chunk)) {
        pack |= 2;
        if (!d.transB) e.N = round_up(d.N, chunk);
        e.ldb = round_up(d.transB ? e.K : e.N, line);
    }
    const int v = pack ? select_variant(e, false) : -1;
    if (v < 0 || !g_variants[v].direct || g_variants[v].kind != KIND_TILED) return false;
    const size_t bytes_a = (pack & 1) ? (size_t)((d.transA ? e.K : d.M) * e.lda * es) : 0;
    const size_t bytes_b = (pack & 2) ? (size_t)((d.transB ? d.N : e.K) * e.ldb * es) : 0;
    const double copy_us = 6.0 + 0.3 * (double)(bytes_a + bytes_b) / 1.0e6;
    const double direct = tiled_cost(g_variants[v], e, choose_split(g_variants[v], e)) + units_of_us(g_variants[v], copy_us);
    const Variant &sv = g_variants[staged];
    const int ss = choose_split(sv, d);
    const bool pays = pack_pays(d, direct, staged_cost(sv, d, ss));
    // in 16 bits also where they pay only against rows that all lie on odd addresses: whether they do is known to the run
    if (!pays && (d.dtype == PEAK_DT_F32 || !pack_pays(d, direct, staged_cost(sv, d, ss, pack & 1 ? 1.67 : 1.0, pack & 2 ? 1.67 : 1.0)))) return false;
    plan_geometry(g, e, v, 0, streamk);
    g->pack = pack;
    g->pack_odd = !pays;
    g->pack_k = e.K; g->pack_m = e.M; g->pack_n = e.N;
    g->pack_ld[0] = e.lda; g->pack_ld[1] = e.ldb;
    g->pack_off[0] = (g->ws_bytes + 255) & ~(size_t)255;    // behind the partials, on 256-byte boundaries
    g->pack_off[1] = (g->pack_off[0] + bytes_a + 255) & ~(size_t)255;
    g->ws_bytes = (g->pack_off[1] + bytes_b + 255) & ~(size_t)255;
    return true;
}

// Selector table from an offline sweep: exact shape -> variant and K split.
struct TuneEntry {
    int dt, ta, tb;
    int64_t M, N, K;
    int variant, split;
};
static std::vector<TuneEntry> g_tuning;
static bool g_tuning_env_done = false;

static int variant_by_name(const char *name)
{
    for (int i = 0; i < NUM_VARIANTS; ++i)
        if (strcmp(g_variants[i].name, name) == 0) return i;
    return -1;
}

// whole decimal number within [lo, hi]; anything else (sign games, overflow, trailing characters) is refused
static bool parse_int(const char *tok, long long lo, long long hi, long long *out)
{
    if (!tok || !*tok) return false;
    char *end = nullptr;
    errno = 0;
    const long long v = strtoll(tok, &end, 10);
    if (errno != 0 || end == tok || *end != 0 || v < lo || v > hi) return false;
    *out = v;
    return true;
}

static int load_tuning_file(const char *path)
{
    FILE *f = fopen(path, "r");
    if (!f) return -1;
    std::vector<TuneEntry> table;
    char line[512];
    bool ok = true;
    while (ok && fgets(line, sizeof line, f)) {
        const size_t len = strlen(line);
        if (len == sizeof line - 1 && line[len - 1] != '\n') { ok = false; break; }   // longer than any valid row
        if (char *hash = strchr(line, '#')) *hash = 0;
        // up to eight whitespace-separated columns; further ones are ignored
        char *tok[8];
        int n = 0;
        for (char *t = strtok(line, " \t\r\n"); t && n < 8; t = strtok(nullptr, " \t\r\n")) tok[n++] = t;
        if (n == 0) continue;                               // blank or comment line
        TuneEntry e;
        long long ta = 0, tb = 0, M = 0, N = 0, K = 0, split = 0;
        ok = n == 8;
        if (ok) {
            e.dt = strcmp(tok[0], "f32") == 0 ? PEAK_DT_F32 : strcmp(tok[0], "f16") == 0 ? PEAK_DT_F16
                 : strcmp(tok[0], "bf16") == 0 ? PEAK_DT_BF16 : -1;
            e.variant = variant_by_name(tok[6]);
            const long long dim_max = (long long)1 << 30;
            ok = e.dt >= 0 && e.variant >= 0 && g_variants[e.variant].dt == e.dt &&
                 parse_int(tok[1], 0, 1, &ta) && parse_int(tok[2], 0, 1, &tb) &&
                 parse_int(tok[3], 1, dim_max, &M) && parse_int(tok[4], 1, dim_max, &N) && parse_int(tok[5], 1, dim_max, &K) &&
                 parse_int(tok[7], 0, 255, &split);
        }
        if (ok) {
            e.ta = (int)ta; e.tb = (int)tb; e.M = M; e.N = N; e.K = K; e.split = (int)split;
            table.push_back(e);
        }
    }
    fclose(f);
    if (!ok) return -1;
    g_tuning.swap(table);
    return (int)g_tuning.size();
}

// The table that ships with the library: peak_gemm_tuning.txt beside the shared object.
static std::string shipped_table_path()
{
    Dl_info info;
    if (!dladdr((const void *)&peak_gemm_variant_count, &info) || !info.dli_fname) return std::string();
    std::string path(info.dli_fname);
    const size_t slash = path.rfind('/');
    path = slash == std::string::npos ? std::string() : path.substr(0, slash + 1);
    return path + "peak_gemm_tuning.txt";
}

static const TuneEntry *tuned(const peak_gemm_desc_t &d)
{
    if (!g_tuning_env_done) {
        g_tuning_env_done = true;
        // PEAK_GEMM_TUNING names another table; set to the empty string it turns the shipped one off
        if (const char *e = getenv("PEAK_GEMM_TUNING")) {
            if (*e) load_tuning_file(e);
        } else {
            const std::string path = shipped_table_path();
            if (!path.empty()) load_tuning_file(path.c_str());
        }
    }
    for (const TuneEntry &e : g_tuning)
        if (e.dt == (int)d.dtype && e.ta == d.transA && e.tb == d.transB && e.M == d.M && e.N == d.N && e.K == d.K &&
            variant_fits(g_variants[e.variant], d))
            return &e;
    return nullptr;
}

int64_t peak::grid_blocks(const Geometry &g)
{
    const int64_t tiles = (int64_t)g.tiles_m * g.tiles_n;
    return g.sk_tiles ? tiles - g.sk_tiles + (int64_t)g.sk_tiles * g.split : tiles * g.split;
}

extern "C" {

int peak_gemm_load_tuning(const char *path)
{
    g_tuning_env_done = true;                               // an explicit call overrides the environment
    if (!path) {
        g_tuning.clear();
        return 0;
    }
    return load_tuning_file(path);
}

const char *peak_status_string(peak_status_t s)
{
    switch (s) {
    case PEAK_OK: return "ok";
    case PEAK_ERR_INVALID_ARG: return "invalid argument";
    case PEAK_ERR_UNSUPPORTED: return "no kernel variant supports this problem";
    case PEAK_ERR_WORKSPACE: return "workspace missing or too small";
    case PEAK_ERR_HIP: return "HIP runtime error at launch";
    case PEAK_ERR_ALLOC: return "host allocation failed";
    }
    return "unknown status";
}

int peak_gemm_variant_count(void) { return NUM_VARIANTS; }

const char *peak_gemm_variant_name(int id)
{
    if (id < 0 || id >= NUM_VARIANTS) return nullptr;
    return g_variants[id].name;
}

peak_status_t peak_gemm_create(const peak_gemm_desc_t *desc, peak_gemm_plan_t **out_plan)
{
    if (out_plan) *out_plan = nullptr;
    if (!desc || !out_plan) return PEAK_ERR_INVALID_ARG;
    const peak_gemm_desc_t &d = *desc;
    if (d.M < 0 || d.N < 0 || d.K < 0) return PEAK_ERR_INVALID_ARG;
    if (d.dtype != PEAK_DT_F32 && d.dtype != PEAK_DT_F16 && d.dtype != PEAK_DT_BF16) return PEAK_ERR_INVALID_ARG;
    if ((d.transA != 0 && d.transA != 1) || (d.transB != 0 && d.transB != 1)) return PEAK_ERR_INVALID_ARG;
    if (d.flags & ~(0xFFFFu | PEAK_GEMM_C_F32 | PEAK_GEMM_STREAMK_ON | PEAK_GEMM_STREAMK_OFF)) return PEAK_ERR_INVALID_ARG;
    if ((d.flags & PEAK_GEMM_STREAMK_ON) && (d.flags & PEAK_GEMM_STREAMK_OFF)) return PEAK_ERR_INVALID_ARG;
    const int64_t min_lda = d.transA ? d.M : d.K, min_ldb = d.transB ? d.K : d.N;
    if (d.lda < (min_lda > 1 ? min_lda : 1) || d.ldb < (min_ldb > 1 ? min_ldb : 1) || d.ldc < (d.N > 1 ? d.N : 1))
        return PEAK_ERR_INVALID_ARG;
    // index arithmetic is 64-bit, but tile counts and the grid are 32-bit
    if (d.M > (int64_t)1 << 30 || d.N > (int64_t)1 << 30 || d.K > (int64_t)1 << 30) return PEAK_ERR_UNSUPPORTED;

    peak_gemm_plan *p = new (std::nothrow) peak_gemm_plan;
    if (!p) return PEAK_ERR_ALLOC;
    memset(p, 0, sizeof *p);
    p->d = d;
    p->g.variant = p->alt.variant = p->small.variant = -1;
    p->g.split = p->alt.split = p->small.split = 1;

    const int forced = (int)(d.flags & 0xFF) - 1;
    const int forced_split = (int)((d.flags >> 8) & 0xFF);

    if (d.M == 0 || d.N == 0 || d.K == 0) {           // nothing to multiply; run() scales C or does nothing
        if (forced >= 0 && (forced >= NUM_VARIANTS || g_variants[forced].dt != d.dtype)) {
            delete p;
            return PEAK_ERR_UNSUPPORTED;
        }
        *out_plan = p;
        return PEAK_OK;
    }

    int pick = -1;
    int table_split = 0;
    bool own_choice = false;                          // neither forced nor from the selector table
    if (forced >= 0) {
        if (forced >= NUM_VARIANTS || !variant_fits(g_variants[forced], d)) {
            delete p;
            return PEAK_ERR_UNSUPPORTED;
        }
        pick = forced;
    } else if (const TuneEntry *t = tuned(d)) {
        pick = t->variant;
        table_split = t->split > 0 ? t->split : -1;
    } else {
        pick = select_variant(d, false);
        own_choice = true;
        if (pick < 0) {
            delete p;
            return PEAK_ERR_UNSUPPORTED;
        }
    }
    // a table entry with split 0 stands for hybrid stream-K
    int streamk = (d.flags & PEAK_GEMM_STREAMK_ON) ? 1 : (d.flags & PEAK_GEMM_STREAMK_OFF) ? -1 : 0;
    if (forced_split <= 0 && streamk == 0 && table_split < 0) streamk = 1;
    plan_geometry(&p->g, d, pick, forced_split > 0 ? forced_split : (table_split > 0 ? table_split : 0), streamk);
    int deep = -1, slices = 0;
    if (own_choice && forced_split <= 0 && p->g.sk_tiles == 0 && deep_split(d, pick, p->g.split, &deep, &slices)) {
        p->small = p->g;
        plan_geometry(&p->g, d, deep, slices);
    }
    // Leading dimensions are known here, base addresses only at run time: a variant that copies
    // 16-byte chunks gets a stand-in that takes any alignment for runs whose A or B base is off that alignment.
    // Such a choice of the cost model's is the stand-in itself where aligned copies are worth making
    // (a table row's variant and split are taken as they are)
    if (own_choice && forced_split <= 0 && !g_variants[pick].direct) {
        Geometry packed = Geometry();
        if (pack_plan(d, pick, &packed, streamk)) {
            p->alt = p->g;
            p->g = packed;
        }
    }
    if (g_variants[pick].direct) {
        const int alt = select_variant(d, true);
        if (alt >= 0) plan_geometry(&p->alt, d, alt, forced_split);
    }
    p->ws_bytes = p->g.ws_bytes > p->alt.ws_bytes ? p->g.ws_bytes : p->alt.ws_bytes;
    if (p->small.ws_bytes > p->ws_bytes) p->ws_bytes = p->small.ws_bytes;
    const int64_t grid = (int64_t)p->g.tiles_m * p->g.tiles_n * p->g.split;   // (an upper bound for a stream-K plan)
    const int64_t grid_alt = p->alt.variant < 0 ? 0 : (int64_t)p->alt.tiles_m * p->alt.tiles_n * p->alt.split;
    if (grid > 0x7FFFFFFF || grid_alt > 0x7FFFFFFF) {
        delete p;
        return PEAK_ERR_UNSUPPORTED;
    }
    *out_plan = p;
    return PEAK_OK;
}

size_t peak_gemm_workspace_bytes(const peak_gemm_plan_t *plan) { return plan ? plan->ws_bytes : 0; }

int peak_gemm_plan_info(const peak_gemm_plan_t *p, char *buf, size_t n)
{
    if (!p) return snprintf(buf, n, "null plan");
    if (p->g.variant < 0)
        return snprintf(buf, n, "variant=none (degenerate size) M=%lld N=%lld K=%lld", (long long)p->d.M,
                        (long long)p->d.N, (long long)p->d.K);
    const Geometry &g = p->g;
    const Variant &v = g_variants[g.variant];
    return snprintf(buf, n,
                    "variant=%d:%s tile=%dx%dx%d threads=%d stages=%d lds=%d split=%d ktiles/slice=%d "
                    "grid=%lld (tiles %dx%d) group_m=%d workspace=%zu unaligned=%s small=%s streamk=%d rot=%d,%d xcdrot=%d pack=%d oddbase=%d acopy=%d",
                    g.variant, v.name, v.bm, v.bn, v.bk, v.nt, v.ns, v.lds, g.split, g.ktiles_per_slice,
                    (long long)grid_blocks(g), g.tiles_m, g.tiles_n, g.group_m, p->ws_bytes,
                    p->alt.variant >= 0 ? g_variants[p->alt.variant].name : "same",
                    p->small.variant >= 0 ? g_variants[p->small.variant].name : "none", g.sk_tiles, g.rot_m, g.rot_n, g.rot_x, g.pack, g.pack_odd,
                    g.a_copy);
}

peak_status_t peak_gemm_destroy(peak_gemm_plan_t *plan)
{
    delete plan;
    return PEAK_OK;
}

}  // extern "C"
