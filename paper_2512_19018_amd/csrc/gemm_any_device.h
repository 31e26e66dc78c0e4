// Tiled kernel with a ring of K tiles on their way into the LDS, every storage type, all four layouts, on the 16x16
// MFMA (16x16x32 for 16-bit operands, 16x16x4 for fp32), in two forms:
//   aligned operands, small tiles ("_m...q<stages>"): for grids that would leave the large tiles' chip idle;
//   operands of any alignment ("_r"): odd leading dimensions, blocks of larger matrices that start anywhere, K that is
//   no whole number of 16-byte chunks.
//
// Both copy global -> LDS directly, 16 bytes per lane: the copies take addresses of any 2-byte alignment (the
// LDS side is always aligned; checked over all of them, rows 16 bytes to 4 KB apart).  Rows along K lie as they do in
// memory, [k][x] rows too, with the transposing read for 16-bit operands.  For operands of any alignment that holds for
// whole K tiles; the tile that K ends in goes through registers, shifted into place (shift_down), and is asked for before the loop.
//
// Bound, 16 bits: the way of the rows into the CU.  72 to 85 bytes per ns and CU where rows start on 128-byte lines, 58 to 68
// where they start anywhere (each piece of a row then lies in one line more than it fills; a sixth less where every other row
// lies on an odd 2-byte address, two fifths less where all do).  fp32: the MFMAs, at 0.75 to 0.9 of their rate.  The any-alignment form went through registers before: 16-byte
// loads, one tile on its way, LDS stores, two barriers' worth of LDS traffic in a chain per tile; more tiles on their way changed nothing.
// Through the ring: fp32 777x1234x1555 TT 42.5 -> 29.5 us, 4095^3 NT 1054 -> 947, 219x1105x1177 NN 16.6 -> 11.0; bf16 704x640x1331 NT 12.0 -> 8.6,
// 407x705x977 TN 11.0 -> 8.6, 1931x1587x1251 TT 28 -> 23.5, 1023x2047x3001 NT 40.8 -> 28.5.
#pragma once

#include "gemm_device.h"

namespace peak {

// WM x WN waves share the tile, WK waves each of its places (the rounds of a stage dealt out over them, their sums
// added in LDS at the end, in wave order); RB: bytes of K per row and stage; EU: waves per SIMD that the register
// budget is cut for; RING: stages in LDS; LOOSE: operands of any alignment.
template <int DT_, bool A_KM_, bool B_KN_, int BM_, int BN_, int WM_, int WN_, int WK_, int RB_, int EU_, int RING_, bool LOOSE_>
struct CfgAny {
    static constexpr int DT = DT_;
    static constexpr bool A_KM = A_KM_, B_KN = B_KN_;
    static constexpr int ESZ = DT_ == DT_F32 ? 4 : 2, EPC = 16 / ESZ;
    static constexpr int FUSED16 = DT_ != DT_F32 ? 1 : 0;   // (see FusedStep)
    static constexpr int BM = BM_, BN = BN_, RB = RB_, CPR = RB_ / 16, BK = RB_ / ESZ;
    static constexpr int WAVES_M = WM_, WAVES_N = WN_, WAVES_K = WK_;
    static constexpr int PLACES = WM_ * WN_, NW = PLACES * WK_, NT = NW * 64;
    static constexpr int WTM = BM / WM_, WTN = BN / WN_, MB = WTM / 16, NB = WTN / 16;
    static constexpr int KROUND = 4 * EPC;                  // k per round of fragment reads: 4 chunks of 16 bytes
    static constexpr int ROUNDS = BK / KROUND / WK_;        // per stage and wave
    static constexpr int EU = EU_, RING = RING_;
    // fp32, any alignment: a sum of its own for every fourth k, where the registers hold them, so that a tile with few waves
    // along K is no further from the exact sum than those of four waves that it stands in for (777x1234x1555 TT, relative error: one
    // sum per wave 5.0e-7 in 64x32 tiles, 3.6e-7 in 32x32 ones; four 2.6e-7 and 1.9e-7; level in time)
    static constexpr int SETS = DT_ == DT_F32 && LOOSE_ && MB * NB <= 4 ? 4 : 1;
    static constexpr bool LOOSE = LOOSE_;
    // fragments of one round at a time, where those of a whole stage do not fit the registers beside the sums (fp32 64x64: 128
    // registers and four workgroups per CU, 148 and three; level with a deep K, K = 59 11.3 us against 13.0 for 8031x467 TT)
    static constexpr bool BY_ROUND = SETS == 4 && EU == 4 && ROUNDS > 1;
    static constexpr int A_BYTES = BM * RB, B_BYTES = BN * RB, STAGE = A_BYTES + B_BYTES;
    static constexpr int RED_BYTES = PLACES * (WK_ - 1) * MB * NB * 1024;
    static constexpr int OUT_BYTES = 32 * (WTN * 4 + 16) * PLACES;        // the turnaround on the way out
    // The least a launch needs, the ring in full, and a launch's own: no more stages than it has K tiles, since with a short K it is
    // the workgroups that share a CU which cover its trips to memory (the whole ring whatever K, and a ring of its K tiles: bf16
    // 5839x5535x43 NT in 128x64 tiles 29.7 us and 24.4, 7795x2115x80 TN 24.8 and 20.3; f16 3848x4144x48 TT in 128x64 ring tiles 14.5
    // and 11.4, 40 aligned products with K to 128 0.875 of the time)
    static constexpr int LDS_LEAST = OUT_BYTES > RED_BYTES ? OUT_BYTES : RED_BYTES;
    static constexpr int LDS_BYTES = RING_ * STAGE > LDS_LEAST ? RING_ * STAGE : LDS_LEAST;
    // Aligned 16-bit tiles below 128x64 keep the whole ring whatever K, as an array of their own: two or three workgroups of them share
    // a CU anyway, and sized by the launch they were 1 % slower (100x4096x4096 11.36 us and 11.25; 60 products of 64x64 tiles 1.3 %).
    static constexpr bool OWN_LDS = !LOOSE_ && DT_ != DT_F32 && BM_ < 128;
    static constexpr int LDS_SHORTEST = OWN_LDS ? 0 : LDS_LEAST;    // 0: the whole ring whatever K
    static int lds_of(int ktiles) { return ktiles >= RING_ ? LDS_BYTES : ktiles * STAGE > LDS_LEAST ? ktiles * STAGE : LDS_LEAST; }
    static_assert(RB_ == 128 || RB_ == 256, "swizzles below");
    static_assert(ROUNDS * WK_ * KROUND == BK && ROUNDS >= 1, "whole rounds per wave");
    static_assert(WTM % 32 == 0 && WTN % 16 == 0, "epilogue slabs of 32 rows");
    static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "whole chunks per thread");
    // rows along K: chunk c of row r at c ^ swizzle(r) (the placement of the 16x16x32 kernels, see Cfg16::swizzle)
    static __device__ __forceinline__ int swizzle(int r)
    {
        if constexpr (RB_ == 128) return ((r >> 1) & 1) | (((r >> 2) & 1) << 2) | (((r >> 3) & 1) << 1);
        else return (r & 1) | (((r >> 1) & 1) << 2) | (((r >> 2) & 1) << 3) | (((r >> 3) & 1) << 1);
    }
    // [k][x] rows of X elements: byte offset of chunk c of k-row k.
    //   16 bits, read four k-rows x 32 bytes per 16 lanes: with rows of 256 bytes and more the placement of the
    //   16x16x32 kernels; with 128-byte rows two neighbouring k-rows share the 256-byte bank period, bit 1 of k
    //   tells the pairs of a read apart and the second term its groups of lanes.
    //   fp32, read one float per lane, k-rows 4 q + e (q = lane / 16) in one read: the four rows go to four 64-byte
    //   groups of banks; with 128-byte rows bits 0 and 2 of k change places, so that rows 4 apart lie next to
    //   each other, and bit 3 picks the half.
    template <int X>
    static __device__ __forceinline__ int kx_offset(int k, int c)
    {
        constexpr int ROWB = X * ESZ;
        static_assert(ROWB >= 128 && (DT_ != DT_F32 || X >= 32), "row sizes of the placements below");
        if constexpr (DT_ == DT_F32) {
            if constexpr (ROWB >= 256) return k * ROWB + ((c ^ (4 * ((k >> 2) & 3))) << 4);
            else return ((k & ~5) | ((k >> 2) & 1) | ((k & 1) << 2)) * ROWB + ((c ^ (4 * ((k >> 3) & 1))) << 4);
        } else {
            const int hi = ((k >> 3) ^ (k >> 4)) & 1;
            if constexpr (ROWB >= 256) return k * ROWB + ((c ^ (4 * (k & 3)) ^ (2 * hi)) << 4);
            else return k * ROWB + ((c ^ (2 * ((k >> 1) & 1)) ^ (4 * hi)) << 4);
        }
    }
    // ... and the other way round: the k-row and chunk whose place is position `pos` of row `slot`
    template <int X>
    static __device__ __forceinline__ void kx_at(int slot, int pos, int &k, int &c)
    {
        k = DT_ == DT_F32 && X * ESZ < 256 ? (slot & ~5) | ((slot >> 2) & 1) | ((slot & 1) << 2) : slot;
        c = pos ^ ((kx_offset<X>(k, 0) >> 4) & (X * ESZ / 16 - 1));
    }
    // fp32: offset of k-row k + e from k-row k, k a multiple of 4
    template <int X>
    static constexpr int kx_step(int e) { return (X * ESZ >= 256 ? e : (e & 2) | (e & 1) << 2) * (X * ESZ); }
};

// Operand of any alignment through registers, one K tile: load asks for it, fix (once it has arrived) shifts the chunks that K
// cuts into place, store writes it where the direct copies would.  Chunks that K or a matrix edge cuts are fetched so that they
// end on the last element: every chunk is one load inside the matrix, also on edge tiles.
// Rows along K: ROWS rows x K.
template <class C, int ROWS>
struct AnyK {
    static constexpr int NCH = ROWS * C::CPR / C::NT;
    const char *panel;                                      // first row, k = 0
    int64_t voff[NCH];                                      // this thread's chunks at k = 0
    int64_t ld, K;
    int rows;                                               // rows of the tile inside the matrix

    PEAK_DEVM void init(const void *base, int64_t ld_, int64_t row0, int64_t nrows, int64_t K_, int tid)
    {
        ld = ld_;
        K = K_;
        rows = nrows - row0 < ROWS ? (int)(nrows - row0) : ROWS;
        panel = (const char *)base + row0 * ld * C::ESZ;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int idx = tid + C::NT * i;
            int row = idx / C::CPR;
            if (row > rows - 1) row = rows - 1;             // duplicate of a valid row; its results are never stored
            voff[i] = (row * ld + (int64_t)(idx % C::CPR) * C::EPC) * C::ESZ;
        }
    }
    // elements by which the fetched chunk lies before its place, in the tile that K ends in
    PEAK_DEVM int back(int64_t k0, int i, int tid) const
    {
        const int over = (int)(k0 - (K - C::EPC)) + (tid + C::NT * i) % C::CPR * C::EPC;
        return over > 0 ? over : 0;
    }
    PEAK_DEVM void load(u32x4 (&v)[NCH], int64_t k0, int tid) const
    {
        const char *p = panel + k0 * C::ESZ;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if (K >= C::EPC) v[i] = load_loose<u32x4, C::ESZ>(p + (voff[i] - back(k0, i, tid) * C::ESZ));
            else v[i] = load_elems<C::DT>(p + voff[i], (int)K - (tid + C::NT * i) % C::CPR * C::EPC);
        }
    }
    PEAK_DEVM void fix(u32x4 (&v)[NCH], int64_t k0, int tid) const
    {
        if (K >= C::EPC) {
#pragma unroll
            for (int i = 0; i < NCH; ++i) v[i] = shift_down<C::DT>(v[i], back(k0, i, tid));
        }
    }
    PEAK_DEVM void store(char *tile, u32x4 (&v)[NCH], int tid) const
    {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int idx = tid + C::NT * i, row = idx / C::CPR;
            *(u32x4 *)(tile + row * C::RB + (((idx % C::CPR) ^ C::swizzle(row)) << 4)) = v[i];
        }
    }
};

// Operand stored as K rows of X.. elements: BK k-rows x COLS.
template <class C, int COLS>
struct AnyX {
    static constexpr int NCH = COLS * C::CPR / C::NT;
    static constexpr int CPX = COLS * C::ESZ / 16;          // chunks per k-row
    const char *base;
    int64_t voff[NCH];
    int shift[NCH];                                         // elements by which the fetched chunk lies before its place
    int64_t ld, K;
    int narrow;                                             // columns of an operand that has fewer than a chunk of them, else 0
    bool edge;                                              // some chunk of the tile is cut by the matrix edge

    PEAK_DEVM void init(const void *base_, int64_t ld_, int64_t x0, int64_t nx, int64_t K_, int tid)
    {
        ld = ld_;
        K = K_;
        base = (const char *)base_;
        narrow = nx < C::EPC ? (int)nx : 0;
        edge = nx - x0 < COLS && !narrow;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int idx = tid + C::NT * i;
            const int64_t x = x0 + (int64_t)(idx % CPX) * C::EPC;
            const int64_t xc = !narrow && x > nx - C::EPC ? nx - C::EPC : x;
            voff[i] = ((idx / CPX) * ld + xc) * C::ESZ;
            shift[i] = (int)(x - xc);
        }
    }
    PEAK_DEVM void load(u32x4 (&v)[NCH], int64_t k0, int tid) const
    {
        const char *p = base + k0 * ld * C::ESZ;
        // k-rows past the end: fetched from the last one, zeroed by fix
        const int last = K - k0 < C::BK ? (int)(K - k0) - 1 : C::BK - 1;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int k = (tid + C::NT * i) / CPX, over = k > last ? k - last : 0;
            const char *src = p + (voff[i] - over * ld * C::ESZ);
            if (!narrow) v[i] = load_loose<u32x4, C::ESZ>(src);
            else v[i] = load_elems<C::DT>(src, narrow - (tid + C::NT * i) % CPX * C::EPC);
        }
    }
    PEAK_DEVM void fix(u32x4 (&v)[NCH], int64_t k0, int tid) const
    {
#pragma unroll
        for (int i = 0; i < NCH; ++i)
            if (K - k0 < C::BK && (tid + C::NT * i) / CPX >= (int)(K - k0)) v[i] = u32x4{0u, 0u, 0u, 0u};
    }
    // (the shift waits until the tile is stored, when the loads have arrived)
    PEAK_DEVM void store(char *tile, u32x4 (&v)[NCH], int tid) const
    {
        if (edge) {
#pragma unroll
            for (int i = 0; i < NCH; ++i) v[i] = shift_down<C::DT>(v[i], shift[i]);
        }
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int idx = tid + C::NT * i;
            *(u32x4 *)(tile + C::template kx_offset<COLS>(idx / CPX, idx % CPX)) = v[i];
        }
    }
};

// Direct copies of [k][x] rows for the ring form: a wave instruction fills 1024 contiguous LDS bytes, which chunk a
// lane fetches makes the placement.  X a whole number of chunks; one at or past the matrix edge fetches the row's last.
template <class C, int COLS>
struct RingX {
    static constexpr int ROWB = COLS * C::ESZ, CPX = ROWB / 16, PER_WAVE = C::BK * ROWB / 1024 / C::NW;
    static_assert(C::BK * ROWB % (1024 * C::NW) == 0 && 64 % CPX == 0, "every wave issues the same number of loads");
    __amdgpu_buffer_rsrc_t rsrc;
    int voff[PER_WAVE], voff_tail[PER_WAVE], step;

    PEAK_DEVM void init(const void *base, int64_t ld, int64_t x0, int64_t nx, int64_t k0, int64_t K, int tail_k, int wave, int lane)
    {
        const uint64_t panel = (uint64_t)((const char *)base + (k0 * ld + x0) * C::ESZ);
        const int64_t bytes = ((K - k0 - 1) * ld + (nx - x0)) * C::ESZ;          // < 2^31, checked when the plan is made
        const uint64_t panel_u = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(panel >> 32)) << 32) |
                                 (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)panel);
        rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)panel_u, 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
        step = __builtin_amdgcn_readfirstlane((int)(C::BK * ld * C::ESZ));
        const int last = (int)((nx - x0) / C::EPC) - 1;
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const int at = (wave + C::NW * i) * 64 + lane;
            int k, c;
            C::template kx_at<COLS>(at / CPX, at % CPX, k, c);
            if (c > last) c = last;
            voff[i] = (int)((k * ld + (int64_t)c * C::EPC) * C::ESZ);
            voff_tail[i] = k >= tail_k ? OOB_VOFFSET : voff[i];
        }
    }
    PEAK_DEVM void issue(char *tile, int ktile, bool tail, int wave) const
    {
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)(tile + (wave + C::NW * i) * 1024),
                                                     16, tail ? voff_tail[i] : voff[i], ktile * step, 0, 0);
    }
};

// Direct copies of operands of any (2-byte) alignment: whole K tiles only, so rows along K need no care.  KX: [k][x] rows.
// A chunk that the matrix edge cuts is copied whole, what lies behind it in memory with it (it feeds columns of C that
// are never stored), so the k-row after it must be the matrix's as well.  The descriptor moves along K with the tiles:
// no limit on the operand's size, but one on its leading dimension.
template <class C, int ROWS, bool KX>
struct RingLoose {
    static constexpr int ROWB = KX ? ROWS * C::ESZ : C::RB, CPX = ROWB / 16;
    static constexpr int PER_WAVE = (KX ? C::BK : ROWS) * ROWB / 1024 / C::NW;
    static_assert((KX ? C::BK : ROWS) * ROWB % (1024 * C::NW) == 0 && 64 % CPX == 0, "every wave issues the same number of loads");
    uint64_t base;
    int64_t step;
    int voff[PER_WAVE];

    static constexpr int64_t LD_LIMIT = ((int64_t)1 << 31) / ((KX ? C::BK : ROWS) * C::ESZ) - ROWB;
    static_assert(((KX ? C::BK : ROWS) - 1) * (LD_LIMIT - 1) * C::ESZ + ROWB < 0x7FFFFFFF, "the last chunk of a tile within 32 bits and the descriptor");
    static PEAK_DEVM bool fits(int64_t ld) { return ld < LD_LIMIT; }
    PEAK_DEVM void init(const void *src, int64_t ld, int64_t x0, int64_t nx, int64_t k0, int wave, int lane)
    {
        const uint64_t first = (uint64_t)((const char *)src + (KX ? k0 * ld + x0 : x0 * ld + k0) * C::ESZ);
        base = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(first >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)first);
        step = KX ? C::BK * ld * C::ESZ : C::RB;
        const int left = nx - x0 < ROWS ? (int)(nx - x0) : ROWS;       // rows or columns of the tile inside the matrix
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const int at = (wave + C::NW * i) * 64 + lane;
            int r = at / CPX, c = at % CPX;
            if constexpr (KX) {
                C::template kx_at<ROWS>(at / CPX, at % CPX, r, c);
                if (c * C::EPC >= left) c = (left - 1) / C::EPC;
            } else {
                c ^= C::swizzle(r);
                if (r > left - 1) r = left - 1;             // duplicate of a valid row; its results are never stored
            }
            voff[i] = (int)((r * ld + (int64_t)c * C::EPC) * C::ESZ);
        }
    }
    PEAK_DEVM void issue(char *tile, int ktile, int wave) const
    {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(base + ktile * step), 0, 0x7FFFFFFF, 0x00020000);
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)(tile + (wave + C::NW * i) * 1024),
                                                     16, voff[i], 0, 0, 0);
    }
};

template <class C>
__global__ __launch_bounds__(C::NT, C::EU) void gemm_any_kernel(const GemmArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the kernel's symbol
    // The launch's C::lds_of(K tiles of a slice) bytes, from address 0 on: the kernel has no other LDS, and in that address space 0 is
    // an address like any other, a null pointer is -1 (hence the bit cast: a cast of the constant 0 would be one).  An extern
    // array's address is known to the assembler only: extra additions, another order of loads and MFMAs, and fp32 64x64 tiles
    // with K of 150 and more 2 % slower.
    __shared__ __attribute__((aligned(1024))) char own[C::OWN_LDS ? C::LDS_BYTES : 1];
    char *const lds = C::OWN_LDS ? own : (char *)__builtin_bit_cast(__attribute__((address_space(3))) char *, 0u);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave_all % C::PLACES, kpar = wave_all / C::PLACES;
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
    const int r16 = lane & 15, q = lane >> 4;

    const int tiles = p.tiles_m * p.tiles_n;
    const int pos = order_of_block(blockIdx.x, tiles * p.split);
    const int slice = __builtin_amdgcn_readfirstlane(quotient((uint32_t)pos, p.by_tiles));
    int tm, tn;
    tile_in_order(p, pos - slice * tiles, tm, tn);
    const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
    const int kt_begin = slice * p.ktiles_per_slice;
    int kt_end = kt_begin + p.ktiles_per_slice;
    if (kt_end > p.ktiles_total) kt_end = p.ktiles_total;
    const int KT = __builtin_amdgcn_readfirstlane(kt_end - kt_begin);   // >= 1 by construction of the plan
    const int64_t kbase = (int64_t)kt_begin * C::BK;

    f32x4 sums[C::SETS][C::MB][C::NB], (&acc)[C::MB][C::NB] = sums[0];
#pragma unroll
    for (int e = 0; e < C::SETS; ++e)
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb) sums[e][mb][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // Fragment addresses of round kpar; round kpar + WAVES_K * i lies a constant on, but for rows along K, whose
    // swizzle does not commute with the chunk number: one address per round of a stage.
    int a_k[C::ROUNDS], b_k[C::ROUNDS], a_x[C::MB], b_x[C::NB];
#pragma unroll
    for (int r = 0; r < C::ROUNDS; ++r) {
        const int c = 4 * (r * C::WAVES_K + kpar) + q, ra = wm * C::WTM + r16, rb = wn * C::WTN + r16;
        a_k[r] = ra * C::RB + ((c ^ C::swizzle(ra)) << 4);
        b_k[r] = C::A_BYTES + rb * C::RB + ((c ^ C::swizzle(rb)) << 4);
    }
    // [k][x] rows.  16 bits: lane i of a group of 16 points at k-row 8 q + i / 4, columns 4 (i % 4) .. + 3 and gets
    // the 4 k of one column; a second read four rows on takes the other half.  fp32: k-rows 4 q + e, column r16.
    auto x_addr = [&](auto xc, int col16) {
        constexpr int X = decltype(xc)::value;
        if constexpr (C::DT == DT_F32) {
            const int col = col16 + r16;
            return C::template kx_offset<X>(kpar * C::KROUND + 4 * q, col >> 2) + (col & 3) * 4;
        } else {
            const int col = col16 + 4 * (r16 & 3);
            return C::template kx_offset<X>(kpar * C::KROUND + 8 * q + (r16 >> 2), col >> 3) + (r16 & 1) * 8;
        }
    };
    if constexpr (C::A_KM) {
#pragma unroll
        for (int i = 0; i < C::MB; ++i) a_x[i] = x_addr(IC<C::BM>{}, wm * C::WTM + i * 16);
    }
    if constexpr (C::B_KN) {
#pragma unroll
        for (int i = 0; i < C::NB; ++i) b_x[i] = C::A_BYTES + x_addr(IC<C::BN>{}, wn * C::WTN + i * 16);
    }
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    auto frag_x = [&](const char *st, int addr, int r, auto xc) -> u32x4 {
        constexpr int X = decltype(xc)::value, ROWB = X * C::ESZ;
        const char *f = st + addr + r * (C::WAVES_K * C::KROUND * ROWB);
        if constexpr (C::DT == DT_F32) {
            return u32x4{*(const uint32_t *)(f + C::template kx_step<X>(0)), *(const uint32_t *)(f + C::template kx_step<X>(1)),
                         *(const uint32_t *)(f + C::template kx_step<X>(2)), *(const uint32_t *)(f + C::template kx_step<X>(3))};
        } else {
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)f);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(f + 4 * ROWB));
            const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
            return u32x4{l2[0], l2[1], h2[0], h2[1]};
        }
    };
    auto frag_a = [&](const char *st, int i, int r) -> u32x4 {
        if constexpr (C::A_KM) return frag_x(st, a_x[i], r, IC<C::BM>{});
        else return *(const u32x4 *)(st + a_k[r] + i * 16 * C::RB);
    };
    auto frag_b = [&](const char *st, int i, int r) -> u32x4 {
        if constexpr (C::B_KN) return frag_x(st, b_x[i], r, IC<C::BN>{});
        else return *(const u32x4 *)(st + b_k[r] + i * 16 * C::RB);
    };

    auto multiply = [&](const u32x4 (&af)[C::MB], const u32x4 (&bf)[C::NB]) {
        // (B's rows feed the instruction's row operand: a lane ends with 4 consecutive n of one m)
        if constexpr (C::DT == DT_F32) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
                    for (int mb = 0; mb < C::MB; ++mb) {
                        const f32x4 b = __builtin_bit_cast(f32x4, bf[nb]), a = __builtin_bit_cast(f32x4, af[mb]);
                        f32x4 &c = sums[e % C::SETS][mb][nb];
                        c = __builtin_amdgcn_mfma_f32_16x16x4f32(b[e], a[e], c, 0, 0, 0);
                    }
        } else {
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
                for (int mb = 0; mb < C::MB; ++mb) {
                    if constexpr (C::DT == DT_BF16)
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bf[nb]),
                                                                              __builtin_bit_cast(bf16x8, af[mb]), acc[mb][nb], 0, 0, 0);
                    else
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, bf[nb]),
                                                                             __builtin_bit_cast(f16x8, af[mb]), acc[mb][nb], 0, 0, 0);
                }
        }
    };

    // Ring form: direct copies, RING - 1 K tiles ahead.  For small tiles the loads' latency is the cost (a 64 x 64 x 64
    // tile's MFMAs take 128 cycles, a trip to the L2 some 500 and to memory over 1500), so most of the CU's LDS holds
    // tiles on their way.  n: K tiles, one at least; issue(kt, stage): the copies of tile kt.
    auto ring_loop = [&](int n, auto &&issue) {
        constexpr int L = (C::A_BYTES + C::B_BYTES) / 1024 / C::NW;      // loads per wave and tile
        static_assert(C::A_BYTES % (1024 * C::NW) == 0 && C::B_BYTES % (1024 * C::NW) == 0, "every wave issues the same number of loads");
        constexpr int P = C::RING - 1;
        static_assert((P - 1) * L < 64, "fits the wait's counter");
        // (the compiler would put a wait for every direct copy in front of a transposing read: assembly, handed over
        // after a wait for everything asked of LDS)
        const uint32_t lds_b0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
        auto tr_read = [&](int addr, auto offc, u32x2 &lo, u32x2 &hi, auto rowbc) {
            constexpr int off = decltype(offc)::value, rowb = decltype(rowbc)::value;
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(off) : "memory");
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(off + 4 * rowb) : "memory");
        };
        auto multiply_stage = [&](int so) {                     // so: the stage's offset in LDS
            const char *st = lds + so;
            if constexpr (C::BY_ROUND) {
                static_for<C::ROUNDS>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    u32x4 af[C::MB], bf[C::NB];
#pragma unroll
                    for (int i = 0; i < C::NB; ++i) bf[i] = frag_b(st, i, r);
#pragma unroll
                    for (int i = 0; i < C::MB; ++i) af[i] = frag_a(st, i, r);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(af, bf);
                    __builtin_amdgcn_sched_barrier(0);
                });
                return;
            }
            u32x4 af[C::ROUNDS][C::MB], bf[C::ROUNDS][C::NB];
            u32x2 al[C::ROUNDS][C::MB], ah[C::ROUNDS][C::MB], bl[C::ROUNDS][C::NB], bh[C::ROUNDS][C::NB];
            constexpr bool TRA = C::A_KM && C::DT != DT_F32, TRB = C::B_KN && C::DT != DT_F32;
            static_for<C::ROUNDS>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                static_for<C::NB>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (TRB) tr_read(lds_b0 + so + b_x[i], IC<r * C::WAVES_K * C::KROUND * C::BN * C::ESZ>{}, bl[r][i], bh[r][i], IC<C::BN * C::ESZ>{});
                    else bf[r][i] = frag_b(st, i, r);
                });
                static_for<C::MB>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (TRA) tr_read(lds_b0 + so + a_x[i], IC<r * C::WAVES_K * C::KROUND * C::BM * C::ESZ>{}, al[r][i], ah[r][i], IC<C::BM * C::ESZ>{});
                    else af[r][i] = frag_a(st, i, r);
                });
            });
            if constexpr (TRA || TRB) {
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, 0));
                static_for<C::ROUNDS>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    if constexpr (TRB) static_for<C::NB>([&](auto ic) {
                        u32x2 &lo = bl[r][decltype(ic)::value], &hi = bh[r][decltype(ic)::value];
                        asm volatile("" : "+v"(lo), "+v"(hi));
                        bf[r][decltype(ic)::value] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                    });
                    if constexpr (TRA) static_for<C::MB>([&](auto ic) {
                        u32x2 &lo = al[r][decltype(ic)::value], &hi = ah[r][decltype(ic)::value];
                        asm volatile("" : "+v"(lo), "+v"(hi));
                        af[r][decltype(ic)::value] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                    });
                });
            }
            __builtin_amdgcn_sched_barrier(0);
            static_for<C::ROUNDS>([&](auto rc) { multiply(af[decltype(rc)::value], bf[decltype(rc)::value]); });
        };
        static_for<P>([&](auto tc) {
            if (decltype(tc)::value < n) issue(decltype(tc)::value, decltype(tc)::value);
        });
        // own copies of tile kt; everybody's, and nobody reads the stage before this one any more; the next copies into that
        int kt = 0;
        for (; kt + C::RING + P <= n; kt += C::RING)
            static_for<C::RING>([&](auto sc) {
                constexpr int s = decltype(sc)::value;
                wait_vmcnt<(P - 1) * L>();
                lds_barrier();
                issue(kt + s + P, (s + P) % C::RING);
                multiply_stage(s * C::STAGE);
            });
        // The last tiles, all of a short K: no copies past the end, fewer behind the one that is waited for.  (Conditions in the
        // loop above cost it 1 to 12 %; the last tile copied again in place of those past it, with one count for all, doubled
        // the copies of a short K: bf16 439x375x131 NN 5.7 us against 4.8.)
        static_for<C::RING + P - 1>([&](auto uc) {
            constexpr int u = decltype(uc)::value, s = u % C::RING;
            if (kt + u < n) {
                const int behind_here = n - 1 - kt - u;
                static_for<P>([&](auto rc) {
                    constexpr int behind = P - 1 - decltype(rc)::value;
                    if (decltype(rc)::value == 0 ? behind_here >= behind : behind_here == behind) wait_vmcnt<behind * L>();
                });
                lds_barrier();
                if (behind_here >= P) issue(kt + u + P, (s + P) % C::RING);
                multiply_stage(s * C::STAGE);
            }
        });
    };
    if constexpr (!C::LOOSE) {
        LoaderDirect<C, C::BM> dA;
        LoaderDirect<C, C::BN> dB;
        RingX<C, C::BM> nA;
        RingX<C, C::BN> nB;
        const int tail_k = __builtin_amdgcn_readfirstlane((int)(p.K - (int64_t)(p.ktiles_total - 1) * C::BK));
        const int tail_tile = tail_k < C::BK ? p.ktiles_total - 1 - kt_begin : -1;   // relative to the slice
        if constexpr (C::A_KM) nA.init(p.A, p.lda, m0, p.a_cols, kbase, p.K, tail_k, wave_all, lane);
        else dA.init(p.A, p.lda, m0, p.M, kbase, p.K, tail_k, wave_all, lane);
        if constexpr (C::B_KN) nB.init(p.B, p.ldb, n0, p.b_cols, kbase, p.K, tail_k, wave_all, lane);
        else dB.init(p.B, p.ldb, n0, p.N, kbase, p.K, tail_k, wave_all, lane);
        int rot = p.rot_x ? (int)((blockIdx.x & 7) * (uint32_t)KT >> 3) : 0;
        if (p.rot_m | p.rot_n) rot = (int)(((int64_t)tn * p.rot_n + (int64_t)tm * p.rot_m + rot) % KT);
        rot = __builtin_amdgcn_readfirstlane(rot);
        auto issue = [&](int kt, int stage) {
            int kr = kt + rot;
            if (kr >= KT) kr -= KT;
            char *st = lds + stage * C::STAGE;
            const bool tail = kr == tail_tile;
            if constexpr (C::A_KM) nA.issue(st, kr, tail, wave_all);
            else dA.template issue<0, 1>(st, kr, tail, wave_all);
            if constexpr (C::B_KN) nB.issue(st + C::A_BYTES, kr, tail, wave_all);
            else dB.template issue<0, 1>(st + C::A_BYTES, kr, tail, wave_all);
        };
        ring_loop(KT, issue);
        if constexpr (C::WAVES_K > 1) lds_barrier();        // everybody's copies, before the sums over waves go through LDS
    } else {
        AnyK<C, C::BM> kA;
        AnyX<C, C::BM> xA;
        AnyK<C, C::BN> kB;
        AnyX<C, C::BN> xB;
        if constexpr (C::A_KM) xA.init(p.A, p.lda, m0, p.M, p.K, tid);
        else kA.init(p.A, p.lda, m0, p.M, p.K, tid);
        if constexpr (C::B_KN) xB.init(p.B, p.ldb, n0, p.N, p.K, tid);
        else kB.init(p.B, p.ldb, n0, p.N, p.K, tid);
        constexpr int CA = AnyK<C, C::BM>::NCH, CB = AnyK<C, C::BN>::NCH;
        auto load = [&](int kt, u32x4 (&a)[CA], u32x4 (&b)[CB]) {
            const int64_t k0 = kbase + (int64_t)kt * C::BK;
            if constexpr (C::A_KM) xA.load(a, k0, tid);
            else kA.load(a, k0, tid);
            if constexpr (C::B_KN) xB.load(b, k0, tid);
            else kB.load(b, k0, tid);
        };
        auto store = [&](char *st, u32x4 (&a)[CA], u32x4 (&b)[CB]) {
            if constexpr (C::A_KM) xA.store(st, a, tid);
            else kA.store(st, a, tid);
            if constexpr (C::B_KN) xB.store(st + C::A_BYTES, b, tid);
            else kB.store(st + C::A_BYTES, b, tid);
        };
        auto fragments = [&](const char *st, int r, u32x4 (&af)[C::MB], u32x4 (&bf)[C::NB]) {
    #pragma unroll
            for (int i = 0; i < C::NB; ++i) bf[i] = frag_b(st, i, r);
    #pragma unroll
            for (int i = 0; i < C::MB; ++i) af[i] = frag_a(st, i, r);
            __builtin_amdgcn_sched_barrier(0);              // (the compiler would sink the reads to their first use)
        };

        // The tile that K ends in (and all tiles of a narrow operand) comes last, through registers; it is asked for first,
        // so that it costs no round trip of its own at the end.
        bool slow = false, cut = false;
        if constexpr (C::A_KM) { slow |= xA.narrow != 0; cut |= xA.edge && p.M % C::EPC != 0; }
        if constexpr (C::B_KN) { slow |= xB.narrow != 0; cut |= xB.edge && p.N % C::EPC != 0; }
        slow |= !(RingLoose<C, C::BM, C::A_KM>::fits(p.lda) && RingLoose<C, C::BN, C::B_KN>::fits(p.ldb));
        // (the direct copies of a cut chunk read on into the next k-row: not on the matrix's last)
        const int64_t whole = slow ? 0 : (p.K - kbase - (cut ? 1 : 0)) / C::BK;
        const int KF = __builtin_amdgcn_readfirstlane((int)(whole < KT ? whole : KT));
        u32x4 ta[CA], tb[CB];
        if (KF < KT) load(KF, ta, tb);
        if (KF > 0) {
            RingLoose<C, C::BM, C::A_KM> rA;
            RingLoose<C, C::BN, C::B_KN> rB;
            rA.init(p.A, p.lda, m0, p.M, kbase, wave_all, lane);
            rB.init(p.B, p.ldb, n0, p.N, kbase, wave_all, lane);
            ring_loop(KF, [&](int kt, int stage) {
                rA.issue(lds + stage * C::STAGE, kt, wave_all);
                rB.issue(lds + stage * C::STAGE + C::A_BYTES, kt, wave_all);
            });
        }
        // After the ring's last barrier every copy has landed and nobody reads the stage after the last tile's any more.
        const int st = (KF % C::RING) * C::STAGE;
        for (int kt = KF; kt < KT; ++kt) {
            const int64_t k0 = kbase + (int64_t)kt * C::BK;
            if constexpr (C::A_KM) xA.fix(ta, k0, tid);
            else kA.fix(ta, k0, tid);
            if constexpr (C::B_KN) xB.fix(tb, k0, tid);
            else kB.fix(tb, k0, tid);
            if (kt > KF) lds_barrier();
            store(lds + st, ta, tb);
            if (kt + 1 < KT) load(kt + 1, ta, tb);
            lds_barrier();
            u32x4 af[C::MB], bf[C::NB];
            static_for<C::ROUNDS>([&](auto rc) {
                fragments(lds + st, decltype(rc)::value, af, bf);
                multiply(af, bf);
            });
        }
        if constexpr (C::WAVES_K > 1) lds_barrier();        // the stages are read, before the sums over waves go through LDS
    }

#pragma unroll
    for (int h = 1; h < C::SETS; h *= 2)                       // pairs, then pairs of pairs
#pragma unroll
        for (int e = 0; e + h < C::SETS; e += 2 * h)
#pragma unroll
            for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < C::NB; ++nb) sums[e][mb][nb] += sums[e + h][mb][nb];

    if constexpr (C::WAVES_K > 1) {
        f32x4 *red = (f32x4 *)lds + lane;
        if (kpar > 0) {
#pragma unroll
            for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < C::NB; ++nb) red[((kpar - 1) * C::PLACES + wave) * (C::MB * C::NB * 64) + (mb * C::NB + nb) * 64] = acc[mb][nb];
        }
        lds_barrier();
        if (kpar > 0) return;
#pragma unroll
        for (int k = 0; k < C::WAVES_K - 1; ++k)
#pragma unroll
            for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < C::NB; ++nb) acc[mb][nb] += red[(k * C::PLACES + wave) * (C::MB * C::NB * 64) + (mb * C::NB + nb) * 64];
    }

    // acc[mb][nb][v] <-> m = 16 mb + lane % 16, n = 16 nb + 4 (lane / 16) + v; slab s = blocks 2 s and 2 s + 1
    auto write_slab = [&](int sl, char *scr) {
        constexpr int SROW = C::WTN * 4 + 16;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb)
                *(f32x4 *)(scr + (16 * h + r16) * SROW + (nb * 16 + 4 * q) * 4) = acc[2 * sl + h][nb];
    };
    auto write16 = [&](int sl, char *scr16, const auto &step) {
        constexpr int SROW16 = C::WTN * 2 + 16;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float x[4 * C::NB];
#pragma unroll
            for (int e = 0; e < 4 * C::NB; ++e) x[e] = acc[2 * sl + h][e / 4][e % 4] * p.alpha;
            if constexpr (!std::is_same_v<std::decay_t<decltype(step)>, NoStep>) step.apply(2 * sl + h, x);
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb) {
                union { u32x2 u; _Float16 hh[4]; __bf16 bb[4]; } pk;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (C::DT == DT_F16) pk.hh[j] = (_Float16)x[4 * nb + j];
                    else pk.bb[j] = (__bf16)x[4 * nb + j];
                }
                *(u32x2 *)(scr16 + (16 * h + r16) * SROW16 + ((nb * 4 + q) ^ h) * 8) = pk.u;
            }
        }
    };
    epilogue_slabs<C, C::WTM / 32>(p, lds, wave, lane, wm, wn, m0, n0, splitk_out(p, slice), write_slab, write16);
#endif
}

}  // namespace peak
