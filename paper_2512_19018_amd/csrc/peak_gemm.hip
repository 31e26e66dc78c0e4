// Device side of the C ABI: the variant table joined from its translation units, the launches,
// the small kernels' instantiations, and the entry point with a workspace of its own.
#include "../../include/peak_gemm.h"

#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>
#include <vector>

#include "gemm_any_device.h"
#include "skinny_device.h"
#include "variant.h"

namespace peak {

// The variant table: the groups of the other translation units, joined in a fixed order.
static const std::vector<Variant> &variants()
{
    static const std::vector<Variant> table = [] {
        std::vector<Variant> t;
        const VariantGroup groups[] = {variants_any_f32(), variants_any_f16(), variants_any_bf16(), variants_bf16_nt(), variants_f16_nt(), variants_bf16_nn(),
                                       variants_f16_nn(),  variants_f32(),     variants_ta(),     variants_skinny(),
                                       variants_mf16(),    variants_mf16t(),   variants_mf16s(),   variants_mf16d(),   variants_mf16r(),
                                       variants_mf16k(),   variants_ring_f32(), variants_ring_f16(), variants_ring_bf16()};
        for (const VariantGroup &g : groups) t.insert(t.end(), g.rows, g.rows + g.count);
        return t;
    }();
    return table;
}

const Variant *planner_variants(int *count)
{
    *count = (int)variants().size();
    return variants().data();
}

int planner_device_cu_count()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
        return v;
    (void)hipGetLastError();
    return 0;
}

}  // namespace peak

using namespace peak;
#define g_variants (variants())

// A stored K x M (at most 64 columns) written out as M rows of K elements (K a whole number of 32), for the streaming
// kernels, which read their small operand along K.  One workgroup turns 64 k-rows around in LDS: reads run along the rows
// of A, writes of 16 bytes along K.  A few MB at most: what it costs is the trips to memory one after the other, so a
// thread's loads go out together (one at a time, with a division for each element's row, bf16 57x14336: 9.2 us against 4.0).
// COLS: columns that the lanes are dealt out over, M rounded up to 4, 16 or 64 (with 64 for all, M = 1 took 1.2 us longer).
template <class T, int COLS>
__global__ __launch_bounds__(256) void stage_a_kernel(const T *A, int64_t lda, T *dst, int M, int64_t K)
{
    constexpr int EPV = 16 / (int)sizeof(T), LPR = 64 / EPV, ROWS = 256 / LPR;   // elements of a store, lanes and rows of a pass
    constexpr int KSTEP = 256 / COLS, LOADS = 64 / KSTEP;
    __shared__ T tile[64][66];
    const int64_t k0 = (int64_t)blockIdx.x * 64;
    const int m = threadIdx.x % COLS, k1 = threadIdx.x / COLS;
    if (m < M) {
        const T *src = A + m;
        T v[LOADS];
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int64_t k = k0 + k1 + KSTEP * i;
            v[i] = src[(k < K ? k : K - 1) * lda];
        }
#pragma unroll
        for (int i = 0; i < LOADS; ++i) tile[k1 + KSTEP * i][m] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < COLS; r += ROWS) {
        const int row = r + threadIdx.x / LPR, k = threadIdx.x % LPR * EPV;
        if (row >= M || k0 + k >= K) continue;
        union { u32x4 u; T e[EPV]; } o;
#pragma unroll
        for (int e = 0; e < EPV; ++e) o.e[e] = tile[k + e][row];
        *(u32x4 *)(dst + (int64_t)row * K + k0 + k) = o.u;
    }
}

template <class T>
static void stage_a(const T *A, int64_t lda, T *dst, int M, int64_t K, dim3 grid, hipStream_t stream)
{
    if (M <= 4) hipLaunchKernelGGL((stage_a_kernel<T, 4>), grid, dim3(256), 0, stream, A, lda, dst, M, K);
    else if (M <= 16) hipLaunchKernelGGL((stage_a_kernel<T, 16>), grid, dim3(256), 0, stream, A, lda, dst, M, K);
    else hipLaunchKernelGGL((stage_a_kernel<T, 64>), grid, dim3(256), 0, stream, A, lda, dst, M, K);
}

// Aligned copies of one or two operands: `rows` rows of `cols` elements at any alignment, written out as `rows_to` rows
// of `ld_to` elements (whole 16-byte chunks, 128-byte lines) with zeros beyond the matrix.  One 16-byte chunk per thread
// and step; A's chunks come first.  Bound by memory: read once, written once.  Every load is a whole chunk inside a row (which
// has one at least), so that a thread's go out together: the chunk that the row's end cuts is the row's last whole one,
// shifted.  With that chunk read element by element behind a branch, a wave that met a row's end - one in two or four - waited
// for each of its loads: the whole product bf16 2049x2047x1031 NT 32.7 us and 29.7, 811x1383x3221 NN 28.9 and 27.0, f16
// 8191x8191x1023 NT 144.7 and 142.1 (eight steps per thread: 30.4, 27.6, 141.9).
struct PackOperand {
    const void *src;
    void *dst;
    int64_t rows, cols, ld, rows_to, ld_to;
};
constexpr int PACK_STEPS = 4;
template <int DT>
__global__ __launch_bounds__(256) void pack_kernel(const PackOperand a, const PackOperand b, int64_t blocks_a)
{
    constexpr int EPC = DT == DT_F32 ? 4 : 8, ESZ = 16 / EPC;
    const bool second = blockIdx.x >= blocks_a;
    const PackOperand &o = second ? b : a;
    const uint32_t per_row = (uint32_t)(o.ld_to / EPC);
    const int64_t total = o.rows_to * per_row;
    const int64_t first = ((int64_t)blockIdx.x - (second ? blocks_a : 0)) * (256 * PACK_STEPS);
    const int64_t r0 = first / per_row;                     // (the workgroup's: the only division in 64 bits)
    const uint32_t c0 = (uint32_t)(first - r0 * per_row) + threadIdx.x;
    u32x4 v[PACK_STEPS];
    uint32_t past[PACK_STEPS];                              // bits of the chunk loaded that lie before the one wanted
#pragma unroll
    for (int s = 0; s < PACK_STEPS; ++s) {
        const uint32_t down = (c0 + 256 * s) / per_row;
        const int64_t r = r0 + down, c = (int64_t)(c0 + 256 * s - down * per_row) * EPC;
        const int64_t from = c + EPC <= o.cols ? c : o.cols - EPC;
        v[s] = load_loose<u32x4, ESZ>((const char *)o.src + ((r < o.rows ? r : o.rows - 1) * o.ld + from) * ESZ);
        past[s] = r < o.rows && c - from < EPC ? (uint32_t)(c - from) * ESZ * 8 : 128;
    }
#pragma unroll
    for (int s = 0; s < PACK_STEPS; ++s) {
        uint64_t lo = v[s][0] | (uint64_t)v[s][1] << 32, hi = v[s][2] | (uint64_t)v[s][3] << 32;
        const uint32_t n = past[s] & 63;
        if (past[s] >= 64) { lo = hi; hi = 0; }
        if (past[s] >= 128) lo = 0;
        lo = lo >> n | (n ? hi << (64 - n) : 0);
        hi >>= n;
        v[s] = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    }
#pragma unroll
    for (int s = 0; s < PACK_STEPS; ++s) {
        const int64_t at = first + threadIdx.x + 256 * s;
        if (at < total) *(u32x4 *)((char *)o.dst + at * 16) = v[s];
    }
}

static int esize_of(int dt) { return dt == PEAK_DT_F32 ? 4 : 2; }
static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

extern "C" {

static peak_status_t run_plan(peak_gemm_plan_t *p, float alpha, const void *A, const void *B, float beta, void *C,
                              const Hook &hook, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!p) return PEAK_ERR_INVALID_ARG;
    const peak_gemm_desc_t &d = p->d;
    if (d.M == 0 || d.N == 0) return PEAK_OK;
    if (!C) return PEAK_ERR_INVALID_ARG;
    const int es = esize_of(d.dtype);
    const int c_dt = (d.flags & PEAK_GEMM_C_F32) ? PEAK_DT_F32 : d.dtype;      // storage type of C
    const int es_c = esize_of(c_dt);
    if ((uintptr_t)C % es_c) return PEAK_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;

    GemmArgs a;
    memset(&a, 0, sizeof a);
    a.A = A; a.B = B; a.C = C; a.ws = nullptr;
    a.M = d.M; a.N = d.N; a.K = d.K;
    a.lda = d.lda; a.ldb = d.ldb; a.ldc = d.ldc;
    a.alpha = alpha; a.beta = beta;
    a.hook = hook;
    a.split = 1;
    if (c_dt != d.dtype) a.flags |= GF_C_F32;

    const bool no_product = (d.K == 0 || alpha == 0.0f);
    if (no_product) {
        if (beta == 1.0f && !(hook.bias_kind | hook.act)) return PEAK_OK;
        const int64_t blocks = cdiv(d.M * d.N, 256);
        if (blocks > 0x7FFFFFFF) return PEAK_ERR_UNSUPPORTED;
        dim3 grid((unsigned)blocks);
        if (c_dt == PEAK_DT_F32) hipLaunchKernelGGL(scale_c_kernel<DT_F32>, grid, dim3(256), 0, stream, a);
        else if (c_dt == PEAK_DT_F16) hipLaunchKernelGGL(scale_c_kernel<DT_F16>, grid, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL(scale_c_kernel<DT_BF16>, grid, dim3(256), 0, stream, a);
        return hipGetLastError() == hipSuccess ? PEAK_OK : PEAK_ERR_HIP;
    }

    if (!A || !B) return PEAK_ERR_INVALID_ARG;
    if ((uintptr_t)A % es || (uintptr_t)B % es) return PEAK_ERR_INVALID_ARG;
    if (p->g.variant < 0) return PEAK_ERR_UNSUPPORTED;

    // (a plan that stages A reads its own aligned copy, whatever the base and rows of A)
    const bool a_al = (uintptr_t)A % 16 == 0 && (d.lda * es) % 16 == 0;
    const bool b_al = (uintptr_t)B % 16 == 0 && (d.ldb * es) % 16 == 0;
    // the selected variant, or its stand-in when it copies 16-byte chunks and a base is off that alignment
    const Geometry *g = &p->g;
    if (g_variants[g->variant].direct && !((a_al || g->a_copy || (g->pack & 1)) && (b_al || (g->pack & 2)))) {
        if (p->alt.variant < 0) return PEAK_ERR_UNSUPPORTED;
        g = &p->alt;
    }
    // (a workspace too small for a deep K split's partials does for the plan with fewer)
    if (g == &p->g && p->small.variant >= 0 && (!workspace || workspace_bytes < g->ws_bytes || (uintptr_t)workspace % 256)) g = &p->small;
    // copies that pay only against rows on odd 2-byte addresses, and none there
    auto odd_rows = [](const void *base, int64_t ld) { return ld % 2 == 0 && (uintptr_t)base % 4 != 0; };
    if (g->pack_odd && !((g->pack & 1) && odd_rows(A, d.lda)) && !((g->pack & 2) && odd_rows(B, d.ldb))) g = &p->alt;
    // (a workspace that does not suit aligned copies, such as the fixed array of peak_gemm_run_static, does for the stand-in)
    if (g->pack && (!workspace || workspace_bytes < g->ws_bytes || (uintptr_t)workspace % 256)) g = &p->alt;
    const Variant &v = g_variants[g->variant];

    if (g->split > 1 || g->a_copy || g->pack) {
        if (!workspace || workspace_bytes < g->ws_bytes) return PEAK_ERR_WORKSPACE;
        if ((uintptr_t)workspace % 256) return PEAK_ERR_INVALID_ARG;
    }
    if (g->split > 1) a.ws = (float *)workspace;
    a.a_cols = d.M; a.b_cols = d.N;
    if (g->pack) {
        PackOperand ops[2] = {};
        const int64_t k_to = g->pack_k;
        if (g->pack & 1) {
            ops[0] = PackOperand{A, (char *)workspace + g->pack_off[0], d.transA ? d.K : d.M, d.transA ? d.M : d.K, d.lda,
                                 d.transA ? k_to : d.M, g->pack_ld[0]};
            a.A = ops[0].dst; a.lda = g->pack_ld[0]; a.a_cols = g->pack_m;
        }
        if (g->pack & 2) {
            ops[1] = PackOperand{B, (char *)workspace + g->pack_off[1], d.transB ? d.N : d.K, d.transB ? d.K : d.N, d.ldb,
                                 d.transB ? d.N : k_to, g->pack_ld[1]};
            a.B = ops[1].dst; a.ldb = g->pack_ld[1]; a.b_cols = g->pack_n;
        }
        a.K = k_to;
        int64_t blocks[2];
        for (int i = 0; i < 2; ++i) blocks[i] = (g->pack >> i) & 1 ? cdiv(ops[i].rows_to * ops[i].ld_to * es / 16, 256 * PACK_STEPS) : 0;
        if (blocks[0] + blocks[1] > 0x7FFFFFFF) return PEAK_ERR_UNSUPPORTED;
        dim3 pgrid((unsigned)(blocks[0] + blocks[1]));
        if (es == 4) hipLaunchKernelGGL(pack_kernel<DT_F32>, pgrid, dim3(256), 0, stream, ops[0], ops[1], blocks[0]);
        else hipLaunchKernelGGL(pack_kernel<DT_F16>, pgrid, dim3(256), 0, stream, ops[0], ops[1], blocks[0]);
        if (hipGetLastError() != hipSuccess) return PEAK_ERR_HIP;
    }
    if (g->a_copy) {
        if (d.M > 64) return PEAK_ERR_UNSUPPORTED;          // (the planner admits no such plan)
        void *copy = (char *)workspace + g->a_copy_off;
        dim3 sgrid((unsigned)cdiv(d.K, 64));
        if (es == 4) stage_a((const uint32_t *)A, d.lda, (uint32_t *)copy, (int)d.M, d.K, sgrid, stream);
        else stage_a((const uint16_t *)A, d.lda, (uint16_t *)copy, (int)d.M, d.K, sgrid, stream);
        if (hipGetLastError() != hipSuccess) return PEAK_ERR_HIP;
        a.A = copy;
        a.lda = d.K;
    }
#ifdef PEAK_TRACE
    // diagnostic build: an unsplit run writes 64 bytes of time stamps per wave into the workspace, if one that large is given
    if (g->split == 1 && workspace && workspace_bytes >= (size_t)g->tiles_m * g->tiles_n * (v.nt / 64) * 64) a.ws = (float *)workspace;
#endif
    set_tile_order(a, g->tiles_m, g->tiles_n, g->group_m);
    a.split = g->split;
    a.ktiles_per_slice = g->ktiles_per_slice;
    a.ktiles_total = g->ktiles_total;
    a.rot_m = g->rot_m;
    a.rot_n = g->rot_n;
    a.rot_x = g->rot_x;
    a.sk_tiles = g->sk_tiles;
    a.by_reduce = divisor((int)cdiv(d.N, REDUCE_COLS));

    int64_t nblocks = grid_blocks(*g);
    if (v.kind == KIND_SKINNY_REG) nblocks = cdiv((int64_t)g->tiles_n * g->split, v.nt / 64);   // one wave per row group and slice
    if (v.launch(a, (unsigned)nblocks, (void *)stream) != 0) return PEAK_ERR_HIP;

    if (g->sk_tiles) {
        // the cut tiles: ordered sum of their slices (the 16x16x32 kernels' tile is 256 x 256)
        dim3 rgrid(256 * (256 / 4) / 256, (unsigned)g->sk_tiles);
        if (c_dt == PEAK_DT_F32 || d.dtype == PEAK_DT_BF16)
            hipLaunchKernelGGL((streamk_reduce_kernel<DT_BF16, 256, 256>), rgrid, dim3(256), 0, stream, a);
        else
            hipLaunchKernelGGL((streamk_reduce_kernel<DT_F16, 256, 256>), rgrid, dim3(256), 0, stream, a);
        if (hipGetLastError() != hipSuccess) return PEAK_ERR_HIP;
    } else if (g->split > 1) {
        dim3 rgrid((unsigned)(cdiv(d.N, REDUCE_COLS) * cdiv(d.M, REDUCE_ROWS)));
        if (c_dt == PEAK_DT_F32) hipLaunchKernelGGL(splitk_reduce_kernel<DT_F32>, rgrid, dim3(256), 0, stream, a);
        else if (c_dt == PEAK_DT_F16) hipLaunchKernelGGL(splitk_reduce_kernel<DT_F16>, rgrid, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL(splitk_reduce_kernel<DT_BF16>, rgrid, dim3(256), 0, stream, a);
        if (hipGetLastError() != hipSuccess) return PEAK_ERR_HIP;
    }
    return PEAK_OK;
}

peak_status_t peak_gemm_run(peak_gemm_plan_t *plan, float alpha, const void *A, const void *B, float beta, void *C,
                            void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_plan(plan, alpha, A, B, beta, C, Hook{nullptr, BIAS_NONE, ACT_NONE}, workspace, workspace_bytes, hip_stream);
}

peak_status_t peak_gemm_run_fused(peak_gemm_plan_t *plan, float alpha, const void *A, const void *B, float beta, void *C,
                                  const peak_gemm_epilogue_t *epilogue,
                                  void *workspace, size_t workspace_bytes, void *hip_stream)
{
    Hook hook{nullptr, BIAS_NONE, ACT_NONE};
    if (epilogue) {
        static_assert(PEAK_BIAS_PER_COLUMN == BIAS_PER_COLUMN && PEAK_BIAS_PER_ROW == BIAS_PER_ROW &&
                      PEAK_ACT_RELU == ACT_RELU && PEAK_ACT_GELU_TANH == ACT_GELU_TANH, "interface and kernel enums agree");
        if (epilogue->bias_kind < PEAK_BIAS_NONE || epilogue->bias_kind > PEAK_BIAS_PER_ROW) return PEAK_ERR_INVALID_ARG;
        if (epilogue->act < PEAK_ACT_NONE || epilogue->act > PEAK_ACT_GELU_TANH) return PEAK_ERR_INVALID_ARG;
        if (epilogue->bias_kind != PEAK_BIAS_NONE) {
            if (!epilogue->bias || (uintptr_t)epilogue->bias % sizeof(float)) return PEAK_ERR_INVALID_ARG;
            hook.bias = (const float *)epilogue->bias;
        }
        hook.bias_kind = epilogue->bias_kind;
        hook.act = epilogue->act;
    }
    return run_plan(plan, alpha, A, B, beta, C, hook, workspace, workspace_bytes, hip_stream);
}

// Workspace of peak_gemm_run_static: one array per GPU, part of the loaded code
// object, held until the process ends.  In host code the array's name only
// stands for the symbol; its address on a device comes from hipGetSymbolAddress
// with that device current.
static __device__ __align__(256) unsigned char scratch[PEAK_GEMM_STATIC_WORKSPACE_BYTES];

constexpr int MAX_DEVICES = 64;
static void *g_scratch_ptr[MAX_DEVICES];          // per device; nullptr until looked up
static std::mutex g_scratch_mutex;

peak_status_t peak_gemm_run_static(peak_gemm_plan_t *plan, float alpha, const void *A, const void *B, float beta,
                                   void *C, void *hip_stream)
{
    if (!plan) return PEAK_ERR_INVALID_ARG;
    // (a plan that would make aligned copies runs its stand-in where the copies do not fit, one with a deep K split that with fewer partials)
    const bool other = plan->g.pack || plan->small.variant >= 0;
    const size_t least = !other ? plan->ws_bytes : plan->alt.ws_bytes > plan->small.ws_bytes ? plan->alt.ws_bytes : plan->small.ws_bytes;
    if (least > (size_t)PEAK_GEMM_STATIC_WORKSPACE_BYTES) return PEAK_ERR_WORKSPACE;
    void *ws = nullptr;
    if (plan->ws_bytes > 0) {
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return PEAK_ERR_HIP;
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void *ptr = nullptr;
            if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
                (void)hipGetLastError();
                return PEAK_ERR_HIP;
            }
            g_scratch_ptr[dev] = ptr;
        }
        ws = g_scratch_ptr[dev];
    }
    // Every element of the partials that the reduction reads is written by the slices of
    // this very call, so nothing of an earlier call's contents needs clearing.
    return run_plan(plan, alpha, A, B, beta, C, Hook{nullptr, BIAS_NONE, ACT_NONE}, ws,
                    ws ? (size_t)PEAK_GEMM_STATIC_WORKSPACE_BYTES : 0, hip_stream);
}

}  // extern "C"
