// Direct 2D image convolution for gfx950 (CDNA4), one tunable configuration
// per compilation. The host library compiles this file at run time with
// hiprtc, once per (configuration, filter size, alignment class), the way the
// paper's tuner compiles each point of its search space (Section 3; the
// convolution's tunable parameters are Table 1).
//
// Computes, for 0 <= y < H, 0 <= x < W (valid cross-correlation, no flip):
//     out[y][x] = sum_{i<FH} sum_{j<FW} in[y+i][x+j] * f[i][j]
// with `in` (H+FH-1) x (W+FW-1), `f` FH x FW, `out` H x W, row-major FP32.
//
// Accumulation order is fixed for every configuration: one FP32 accumulator
// per output, fused multiply-add, taps in i-ascending then j-ascending order.
// Every configuration (and the batched kernel) therefore returns the same
// bits for the same inputs.
//
// Compile-time parameters (-D):
//   CONV_BX, CONV_BY   workgroup shape in threads (block_size_x / block_size_y)
//   CONV_TX, CONV_TY   outputs per thread along x and y (tile_size_x / _y)
//   CONV_USE_LDS       1: the workgroup stages its input halo tile in LDS
//   CONV_FCONST        1: filter copied into this module's __constant__ array
//                      0: filter read through a const __restrict__ pointer
//   CONV_UNROLL        unroll of the input-row loop (0 = full)
//   CONV_FH, CONV_FW   filter size
//   CONV_VIN           input vector width 1/2/4
//   CONV_VOUT          output vector width 1/2/4
//                      The library builds every kernel with 4 and 4, for rows
//                      of any width: a gfx9-family access of several dwords
//                      needs only dword alignment in the alignment mode the
//                      ROCm driver sets, and a raw buffer load checks each
//                      dword against the buffer size (a vector that straddles
//                      the end of the input reads zeros past it).
//   CONV_NAME          kernel symbol (one per configuration, so that profiles
//                      tell configurations apart); default conv2d_direct
//   CONV_BATCH         1: build the batched kernel (many images of
//                      one filter size, described in device memory) instead
//
// Design (MI355X):
//  * Each thread owns a TY x TX register tile of outputs, contiguous in x.
//    It walks the TY+FH-1 input rows its tile needs once each: a row window of
//    TX+FW-1 values is loaded into VGPRs and feeds every output row that uses
//    it (TY*TX*FW FMAs per window in the steady state). Filter taps are wave
//    uniform and are read with scalar loads, so each FMA is
//    v_fmac_f32 acc, s_tap, v_in.
//  * With an unroll other than 1 and tiles of whole 2 x 2 output blocks, most
//    of those FMAs run on the matrix cores instead, at twice the rate and with
//    the same bits (MatrixRows below).
//  * Global reads use raw buffer loads: an out-of-range dword reads 0
//    instead of faulting, so edge tiles need no clamping; outputs outside the
//    image are simply not stored.
//  * Workgroup ids are remapped so that each of the 8 XCDs (dispatched
//    round-robin) receives one contiguous run of tiles, keeping vertically
//    adjacent tiles, which share FH-1 input rows, in the same L2.

#ifndef CONV_BATCH
#define CONV_BATCH 0
#endif

#ifndef CONV_BX
#error "CONV_BX must be defined"
#endif

#ifndef CONV_NAME
#define CONV_NAME conv2d_direct
#endif

typedef unsigned int u32;
typedef u32 u32x2 __attribute__((ext_vector_type(2)));
typedef u32 u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The CPU build of this file has no matrix instruction unless its harness
// supplies one under the builtin's name (and says so).
#if defined(__AMDGCN__) || defined(CONV_EMULATED_MFMA)
#define CONV_HAVE_MFMA 1
#else
#define CONV_HAVE_MFMA 0
#endif
// Where the matrix path is possible but slower (Geo::PAYS_LDS, PAYS_GLOBAL), the
// plain one runs; the CPU harness takes it wherever it is possible.
#if defined(CONV_EMULATED_MFMA)
#define CONV_MATRIX_PAYS true
#else
#define CONV_MATRIX_PAYS (LDS ? PAYS_LDS : PAYS_GLOBAL)
#endif

// At least two waves per SIMD on the matrix path: with more than 256 registers
// to hand out, the compiler keeps the accumulators of matrix instructions in
// the other half of the register file, where plain FMAs cannot reach them, and
// moves each one out and back around every FMA.
#if defined(__AMDGCN__)
#define CONV_WAVES __attribute__((amdgpu_waves_per_eu(G1::MATRIX ? 2 : 1)))
#else
#define CONV_WAVES
#endif

static constexpr int gcd4(int t) { return (t % 4 == 0) ? 4 : ((t % 2 == 0) ? 2 : 1); }
static constexpr int min_(int a, int b) { return a < b ? a : b; }

// Derived sizes of one configuration (filter FH x FW, workgroup BX x BY
// threads, TX x TY outputs per thread, LDS staging on/off, row-loop unroll,
// input/output vector widths).
template <int FH, int FW, int BX, int BY, int TX, int TY, int LDS, int UNROLL, int VIN, int VOUT>
struct Geo {
    static constexpr int NT = BX * BY;
    static constexpr int WIN = TX + FW - 1;      // input values a thread's row window needs
    static constexpr int NROWS = TY + FH - 1;    // input rows a thread walks
    // Vector width of a thread's window loads: min(gcd(TX, 4), VIN) from
    // global memory, gcd(TX, 4) from LDS (pitch a multiple of 4, the window
    // starting at a multiple of TX, so LDS reads stay aligned). The register
    // window is padded to a whole number of those vectors.
    static constexpr int WVEC = LDS ? gcd4(TX) : min_(gcd4(TX), VIN);
    static constexpr int WIN_PAD = ((WIN + WVEC - 1) / WVEC) * WVEC;
    static constexpr int SVEC = min_(gcd4(TX), VOUT);   // output store width
    // Input halo tile of one workgroup in LDS, rows x pitch floats. The pitch
    // is padded to a multiple of 4 (aligned ds_read_b128) plus 4 when it would
    // otherwise be a multiple of 32 banks' worth, to spread the rows a wave
    // reads over banks.
    static constexpr int LDS_ROWS = BY * TY + FH - 1;
    static constexpr int LDS_COLS = BX * TX + FW - 1;
    static constexpr int LDS_CHUNKS = (LDS_COLS + VIN - 1) / VIN;
    static constexpr int LDS_PITCH0 = ((LDS_CHUNKS * VIN + 3) / 4) * 4;
    static constexpr int LDS_PITCH = (LDS_PITCH0 % 32 == 0) ? LDS_PITCH0 + 4 : LDS_PITCH0;
    static constexpr int LDS_FLOATS = LDS ? LDS_ROWS * LDS_PITCH : 4;
    static constexpr int ROW_UNROLL = UNROLL == 0 ? NROWS : UNROLL;   // 0 = the whole row loop
    // Where the matrix path is the faster one. With the tile in LDS it is from 3
    // x 3 on (4 x (9 FMAs) there take 144 cycles plain and 4 * 8 + 20 * 4 = 112
    // on it, 17 x 17 4624 and 2576), but not for 2 x 2 outputs under a tall
    // filter, whose rows hold too few interior columns for the load of their
    // taps (31 x 3 at 4096 x 4096: 55 and 67 us rolled, fully unrolled 75 and 71
    // but 4.6 and 5.6 at 700 x 700).
    static constexpr bool PAYS_LDS = TX * TY >= 8 || FH <= 4 * FW;
    // Without LDS a thread reads its window from global memory row by row, and
    // small tiles under small filters are bound by those loads, to which the
    // path adds that of the taps. Measured at 4096 x 4096, plain and matrix: 2 x
    // 2 outputs 3 x 3 19.5 and 26.3 us, 9 x 9 61 and 73, 17 x 17 172 and 197
    // (but 297 and 197 fully unrolled, where the taps no longer fit the scalar
    // registers); 4 x 2 7 x 7 29 and 34, 9 x 9 equal, 11 x 11 61 and 59; 4 x 4
    // 5 x 5 fully unrolled 20.2 and 22.1, unroll 2 24.0 and 22.2, 31 x 3 61 and
    // 68, 9 x 9 41 and 32.
    static constexpr int SIDE = min_(FH, FW);
    static constexpr bool PAYS_GLOBAL = TX * TY >= 16 && SIDE >= 9   ? true
                                        : TX >= 4 && TY >= 4         ? UNROLL != 0 && FH <= 4 * FW
                                        : TX * TY >= 8               ? SIDE >= 11
                                                                     : SIDE >= 15 && UNROLL == 0;
    // Matrix path (see MatrixRows): whole waves, output tiles of whole 2 x 2
    // blocks, a filter with interior taps, and a row loop that is not asked to
    // stay rolled (unroll 1 keeps one row's plain FMAs as its body).
    static constexpr bool MATRIX = CONV_HAVE_MFMA && UNROLL != 1 && TX % 2 == 0 && TY % 2 == 0 && NT % 64 == 0 &&
                                   FH >= 3 && FW >= 3 && CONV_MATRIX_PAYS;
};

// Filter taps: the module's __constant__ copy, or the filter pointer.
#if CONV_FCONST
__constant__ float conv_filter[CONV_FH * CONV_FW];
#define TAPS conv_filter
#else
#define TAPS filt
#endif

// Pointers that come out of a descriptor could point anywhere as far as the
// compiler knows; it reads and writes through them with flat accesses, the taps
// by vector loads in every row. Constant memory for the taps gives scalar loads,
// global memory for the outputs plain stores.
#if CONV_BATCH && defined(__AMDGCN__)
typedef const __attribute__((address_space(4))) float* TapPtr;
#define CONV_GLOBAL __attribute__((address_space(1)))
#else
typedef const float* __restrict__ TapPtr;
#define CONV_GLOBAL
#endif

static __device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const float* p, u32 bytes)
{
    // Word 3 = 0x00020000: raw (untyped) dword access, the gfx9-family value.
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)bytes, 0x00020000);
}

// Loads N consecutive floats from byte offset `off` of the buffer into dst[0..N).
// Whole vectors are bit-cast: bit-casting a single ext-vector element
// (v.y, ...) is miscompiled by this clang into a read of element 0.
template <int V, int N>
static __device__ __forceinline__ void buffer_row(float* dst, __amdgpu_buffer_rsrc_t rs, u32 off)
{
#pragma unroll
    for (int m = 0; m < N; m += V) {
        if constexpr (V == 4) {
            f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off + 4u * m), 0, 0));
            dst[m + 0] = v.x;
            dst[m + 1] = v.y;
            dst[m + 2] = v.z;
            dst[m + 3] = v.w;
        } else if constexpr (V == 2) {
            f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(off + 4u * m), 0, 0));
            dst[m + 0] = v.x;
            dst[m + 1] = v.y;
        } else {
            u32 v = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(off + 4u * m), 0, 0);
            dst[m] = __builtin_bit_cast(float, v);
        }
    }
}

// Loads N consecutive floats from LDS (V-element aligned) into dst[0..N).
template <int V, int N>
static __device__ __forceinline__ void lds_row(float* dst, const float* src)
{
#pragma unroll
    for (int m = 0; m < N; m += V) {
        if constexpr (V == 4) {
            f32x4 v = *(const f32x4*)(src + m);
            dst[m + 0] = v.x; dst[m + 1] = v.y; dst[m + 2] = v.z; dst[m + 3] = v.w;
        } else if constexpr (V == 2) {
            f32x2 v = *(const f32x2*)(src + m);
            dst[m + 0] = v.x; dst[m + 1] = v.y;
        } else {
            dst[m] = src[m];
        }
    }
}

// Workgroup id -> tile id: XCD x (= id mod 8) gets the contiguous tile range
// [start(x), start(x) + count(x)); a bijection on [0, n_tiles).
static __device__ __forceinline__ int xcd_remap(int id, int n_tiles)
{
    const int q = n_tiles >> 3, rem = n_tiles & 7;
    const int xcd = id & 7, k = id >> 3;
    return xcd * q + min_(xcd, rem) + k;
}

#if CONV_HAVE_MFMA
// The rows of a thread's tile on the matrix cores.
//
// v_mfma_f32_4x4x1_16b adds, in each of 16 blocks of 4 lanes, the product of a
// 4-vector A and a 4-vector B to a 4 x 4 matrix; lane l of a block keeps
// column l of it in 4 registers and supplies B[l]. So with B = one input value
// of the lane's own window, the instruction is 4 FMAs of that value into 4
// accumulators of the same lane, acc[m] += A[m] * w: the outputs of a 2 x 2
// block (rows y, y+1, columns x, x+1) with the four taps
// f[i - my][k - mx] that input value w[i][k] meets there, m = 2 my + mx. Every
// such product is one the convolution needs where i is in [1, FH-1] and k in
// [1, FW-1]; the rim of the (FH+1) x (FW+1) inputs of a 2 x 2 block stays on
// plain FMAs, so that no product with a padding zero is added (an infinity in
// the input reaches only the outputs it belongs to) and every output still
// sums its taps one by one in the fixed order, in FMAs that round alike: the
// bits are those of the plain path.
//
// A needs no broadcast code: one register holds the four taps of 16 columns k
// (lane 4 q + m: column 1 + q), and the instruction's broadcast control
// (cbsz 4, abid q) feeds block q's taps to all blocks. A filter row pair thus
// costs one register per 16 columns, gathered from the filter by one load.
//
// 4 x 4 x 1 runs 256 FMAs in 8 cycles, a plain FMA 64 in 4: a 17 x 17 block
// takes 256 * 8 + 132 * 4 = 2576 cycles against 1156 * 4 = 4624 (the two do
// not overlap: a mix of both measured the sum of their times). Bound by these
// issue cycles: at 4096 x 4096 / 17 x 17 they are 171 of the 184 thousand
// cycles a CU is busy. Measured against the plain path's winners, 4096 x 4096:
// 31 x 31 432 -> 256 us, 17 x 17 134.7 -> 88.1 (110 TFLOP/s), 15 x 15 106 ->
// 73, 9 x 9 42 -> 34, 7 x 7 27.6 -> 25.8 and 3 x 3 21.8 -> 19.3 (both then near
// what their 134 MB take: 28 us at the rate of a large copy).
template <int FH, int FW, int TX, int TY, class G>
struct MatrixRows {
    static constexpr int NG = TX / 2, NP = TY / 2;    // 2 x 2 blocks along x and y
    static constexpr int NA = (FW - 1 + 15) / 16;     // tap registers per filter row pair
    // Rows in which every block row is inside the filter: [FIRST, LAST].
    static constexpr int FIRST = 2 * NP - 1, LAST = FH - 1;
    // With the row loop fully unrolled and few enough of them, all taps are
    // loaded once, ahead of the tile (`held`); else each row loads its own.
    static constexpr bool HOLD = G::ROW_UNROLL >= G::NROWS && NA * (FH - 1) <= 32;

    f32x4 acc[NP][NG];
    float held[HOLD ? FH - 1 : 1][NA];

    // The taps of filter rows i (my = 0) and i - 1 (my = 1).
    template <class Rsrc>
    static __device__ __forceinline__ void taps(float (&a)[NA], Rsrc rf, u32 lane_off, int i)
    {
#pragma unroll
        for (int n = 0; n < NA; ++n)
            a[n] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                 rf, (int)(lane_off + (u32)((i - 1) * FW + 16 * n) * 4u), 0, 0));
    }

    // Is block row p at an input row r that meets interior taps (r is a
    // constant after unrolling, or any row of the steady range)?
    static __device__ __forceinline__ constexpr bool inside(int p, int r) { return r - 2 * p >= 1 && r - 2 * p < FH; }

    // The interior columns of input row r, for every block row inside.
    template <bool STEADY, int N, int K>
    __device__ __forceinline__ void columns(int r, const float (&a)[NP][NA], const float* w)
    {
        if constexpr (K < 16 && 16 * N + K < FW - 1) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (STEADY || inside(p, r)) {
#pragma unroll
                    for (int g = 0; g < NG; ++g)
                        acc[p][g] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[p][N], w[2 * g + 1 + 16 * N + K], acc[p][g],
                                                                       4, K, 0);
                }
            columns<STEADY, N, K + 1>(r, a, w);
        } else if constexpr (K == 16 && N + 1 < NA) {
            columns<STEADY, N + 1, 0>(r, a, w);
        }
    }

    // Block row p's first (MY = 0, filter row 0) or last input row (MY = 1,
    // filter row FH - 1): one output row of the two, plain FMAs.
    template <int MY>
    __device__ __forceinline__ void rim(int p, const float* w, TapPtr ft)
    {
#pragma unroll
        for (int j = 0; j < FW; ++j) {
            const float fv = ft[(MY ? (FH - 1) * FW : 0) + j];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                acc[p][g][2 * MY] = __builtin_fmaf(w[2 * g + j], fv, acc[p][g][2 * MY]);
                acc[p][g][2 * MY + 1] = __builtin_fmaf(w[2 * g + 1 + j], fv, acc[p][g][2 * MY + 1]);
            }
        }
    }

    // Column k = 0 (FIRSTCOL) or FW of block row p at its input row i.
    template <bool FIRSTCOL>
    __device__ __forceinline__ void side(int p, int i, const float* w, TapPtr ft)
    {
        constexpr int J = FIRSTCOL ? 0 : FW - 1, K = FIRSTCOL ? 0 : FW, X = FIRSTCOL ? 0 : 1;
        const float f0 = ft[i * FW + J], f1 = ft[(i - 1) * FW + J];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            acc[p][g][X] = __builtin_fmaf(w[2 * g + K], f0, acc[p][g][X]);
            acc[p][g][2 + X] = __builtin_fmaf(w[2 * g + K], f1, acc[p][g][2 + X]);
        }
    }

    // Input row r (a constant after unrolling, unless STEADY) for every block
    // row. The plain FMAs of a row come in one run, the matrix instructions in
    // another, and the scheduler keeps them so: each change from one to the
    // other and back costs about 6 cycles (14 cycles for one of each become
    // 21 when they alternate).
    template <bool STEADY, class Rsrc>
    __device__ __forceinline__ void row(int r, const float* w, Rsrc rf, u32 lane_off, TapPtr ft)
    {
        constexpr int kFence = 0x4 | 0x10 | 0x80;   // scalar and memory instructions may cross, ALU ones not
        float a[NP][NA];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int i = r - 2 * p;
            if (STEADY || inside(p, r)) {
                if constexpr (HOLD) {
#pragma unroll
                    for (int n = 0; n < NA; ++n)
                        a[p][n] = held[i - 1][n];
                } else {
                    taps(a[p], rf, lane_off, i);
                }
                side<true>(p, i, w, ft);
            } else if (i == 0) {
                rim<0>(p, w, ft);
            } else if (i == FH) {
                rim<1>(p, w, ft);
            }
        }
        __builtin_amdgcn_sched_barrier(kFence);
        columns<STEADY, 0, 0>(r, a, w);
        __builtin_amdgcn_sched_barrier(kFence);
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (STEADY || inside(p, r))
                side<false>(p, r - 2 * p, w, ft);
    }
};
#endif

// One output tile of (BY*TY) x (BX*TX) at tile coordinates (tile_y, tile_x)
// of an image. Every thread of the workgroup calls it (the LDS variant
// contains a barrier). `lds` is the workgroup's LDS tile.
template <int FH, int FW, int BX, int BY, int TX, int TY, int LDS, int UNROLL, int VIN, int VOUT>
static __device__ __forceinline__ void conv_tile(const float* __restrict__ in, const float* __restrict__ filt,
                                                 float* __restrict__ out, int H, int W, u32 in_bytes,
                                                 int tile_x, int tile_y, float* __restrict__ lds)
{
    using G = Geo<FH, FW, BX, BY, TX, TY, LDS, UNROLL, VIN, VOUT>;
    int tid = (int)threadIdx.x;
#if CONV_BATCH && defined(__AMDGCN__)
    // Keeps what depends on the thread inside the batched kernel's tile loop,
    // which nearly always runs once: hoisted out, it held 26 registers at 17 x
    // 17.
    asm volatile("" : "+v"(tid));
#endif
    const int lx = tid % BX;
    const int ly = tid / BX;
    const int x0 = tile_x * (BX * TX) + lx * TX;
    const int y0 = tile_y * (BY * TY) + ly * TY;
    const u32 P = (u32)W + (FW - 1);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(in, in_bytes);
    TapPtr const taps = (TapPtr)TAPS;

#if CONV_HAVE_MFMA
    using M = MatrixRows<FH, FW, TX, TY, G>;
    M m;
    const u32 lane = (u32)tid & 63u;
    const u32 lane_off = ((1u - ((lane >> 1) & 1u)) * FW + (lane >> 2) + 1u - (lane & 1u)) * 4u;
    const __amdgpu_buffer_rsrc_t rf = make_rsrc(filt, FH * FW * 4u);
    if constexpr (G::MATRIX && M::HOLD) {
#pragma unroll
        for (int i = 1; i < FH; ++i)
            M::taps(m.held[i - 1], rf, lane_off, i);
    }
#endif

    const float* lbase = lds;
    if constexpr (LDS) {
        // The halo tile, chunk by chunk in row order, NT chunks at a time. The
        // loads of STAGE steps are in flight together (one exposed memory
        // latency instead of one per step), and a step moves every thread by
        // the same number of rows and chunks, so positions are only added up.
        constexpr int STEPS = (G::LDS_ROWS * G::LDS_CHUNKS + G::NT - 1) / G::NT;
        constexpr int STAGE = min_(STEPS, 8);
        constexpr int DR = G::NT / G::LDS_CHUNKS, DC = G::NT % G::LDS_CHUNKS;
        int c = tid;
        int cc = c % G::LDS_CHUNKS, rr = c / G::LDS_CHUNKS;
        u32 off = (((u32)tile_y * (BY * TY) + (u32)rr) * P + (u32)tile_x * (BX * TX) + (u32)(cc * VIN)) * 4u;
        float* dst = lds + rr * G::LDS_PITCH + cc * VIN;
        const u32 step = ((u32)DR * P + (u32)(DC * VIN)) * 4u;
        const u32 wrap = (P - (u32)(G::LDS_CHUNKS * VIN)) * 4u;
        auto advance = [&] {
            c += G::NT;
            cc += DC;
            off += step;
            dst += DR * G::LDS_PITCH + DC * VIN;
            if (DC != 0 && cc >= G::LDS_CHUNKS) {
                cc -= G::LDS_CHUNKS;
                off += wrap;
                dst += G::LDS_PITCH - G::LDS_CHUNKS * VIN;
            }
        };
#pragma unroll 1
        for (int s0 = 0; s0 < STEPS; s0 += STAGE) {
            float v[STAGE][VIN];
            float* to[STAGE];
#pragma unroll
            for (int s = 0; s < STAGE; ++s) {
                to[s] = c < G::LDS_ROWS * G::LDS_CHUNKS ? dst : nullptr;
                buffer_row<VIN, VIN>(v[s], rs, off);
                advance();
            }
#pragma unroll
            for (int s = 0; s < STAGE; ++s) {
                if (to[s]) {
                    if constexpr (VIN == 4) {
                        *(f32x4*)to[s] = f32x4{v[s][0], v[s][1], v[s][2], v[s][3]};
                    } else {
#pragma unroll
                        for (int m = 0; m < VIN; ++m)
                            to[s][m] = v[s][m];
                    }
                }
            }
        }
        __syncthreads();
        lbase = lds + (ly * TY) * G::LDS_PITCH + lx * TX;
    }

    const u32 off0 = ((u32)y0 * P + (u32)x0) * 4u;
    float acc[TY][TX];

#if CONV_HAVE_MFMA
    if constexpr (G::MATRIX) {
        // Matrix instructions take their A operand from lanes that may lie
        // outside the image, so a wave computes with all of its lanes or not
        // at all; what outside lanes read is in range or zero, and unused.
        if (__builtin_amdgcn_ballot_w64(x0 < W && y0 < H) == 0)
            return;
#pragma unroll
        for (int p = 0; p < M::NP; ++p)
#pragma unroll
            for (int g = 0; g < M::NG; ++g)
                m.acc[p][g] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        auto window = [&](float* w, int r) {
            if constexpr (LDS)
                lds_row<G::WVEC, G::WIN_PAD>(w, lbase + r * G::LDS_PITCH);
            else
                buffer_row<G::WVEC, G::WIN_PAD>(w, rs, off0 + (u32)r * P * 4u);
        };
        if constexpr (M::FIRST <= M::LAST && G::ROW_UNROLL < G::NROWS) {
#pragma unroll
            for (int r = 0; r < M::FIRST; ++r) {
                float w[G::WIN_PAD];
                window(w, r);
                m.template row<false>(r, w, rf, lane_off, taps);
            }
#pragma unroll G::ROW_UNROLL
            for (int r = M::FIRST; r <= M::LAST; ++r) {
                float w[G::WIN_PAD];
                window(w, r);
                m.template row<true>(r, w, rf, lane_off, taps);
            }
#pragma unroll
            for (int r = M::LAST + 1; r < G::NROWS; ++r) {
                float w[G::WIN_PAD];
                window(w, r);
                m.template row<false>(r, w, rf, lane_off, taps);
            }
        } else {
#pragma unroll
            for (int r = 0; r < G::NROWS; ++r) {
                float w[G::WIN_PAD];
                window(w, r);
                m.template row<false>(r, w, rf, lane_off, taps);
            }
        }
#pragma unroll
        for (int o = 0; o < TY; ++o)
#pragma unroll
            for (int k = 0; k < TX; ++k)
                acc[o][k] = m.acc[o / 2][k / 2][2 * (o & 1) + (k & 1)];
        if (x0 >= W || y0 >= H)
            return;
    } else
#endif
    {
    if (x0 >= W || y0 >= H)
        return;

#pragma unroll
    for (int o = 0; o < TY; ++o)
#pragma unroll
        for (int k = 0; k < TX; ++k)
            acc[o][k] = 0.0f;

#pragma unroll G::ROW_UNROLL
    for (int r = 0; r < G::NROWS; ++r) {
        float w[G::WIN_PAD];
        if constexpr (LDS)
            lds_row<G::WVEC, G::WIN_PAD>(w, lbase + r * G::LDS_PITCH);
        else
            buffer_row<G::WVEC, G::WIN_PAD>(w, rs, off0 + (u32)r * P * 4u);
#pragma unroll
        for (int o = 0; o < TY; ++o) {
            const int i = r - o;
            if (i >= 0 && i < FH) {
#pragma unroll
                for (int j = 0; j < FW; ++j) {
                    const float fv = taps[i * FW + j];
#pragma unroll
                    for (int k = 0; k < TX; ++k)
                        acc[o][k] = __builtin_fmaf(w[k + j], fv, acc[o][k]);
                }
            }
        }
    }
    }

#pragma unroll
    for (int o = 0; o < TY; ++o) {
        const int y = y0 + o;
        if (y < H) {
            CONV_GLOBAL float* orow = (CONV_GLOBAL float*)out + (size_t)y * (size_t)W + x0;
            if (x0 + TX <= W) {
#pragma unroll
                for (int k = 0; k < TX; k += G::SVEC) {
                    if constexpr (G::SVEC == 4) {
                        f32x4 v = {acc[o][k], acc[o][k + 1], acc[o][k + 2], acc[o][k + 3]};
                        __builtin_nontemporal_store(v, (CONV_GLOBAL f32x4*)(orow + k));
                    } else if constexpr (G::SVEC == 2) {
                        f32x2 v = {acc[o][k], acc[o][k + 1]};
                        __builtin_nontemporal_store(v, (CONV_GLOBAL f32x2*)(orow + k));
                    } else {
                        __builtin_nontemporal_store(acc[o][k], orow + k);
                    }
                }
            } else {
#pragma unroll
                for (int k = 0; k < TX; ++k)
                    if (x0 + k < W)
                        orow[k] = acc[o][k];
            }
        }
    }
}

#if CONV_BATCH == 0
// One image: one workgroup per tile, tiles_x * tiles_y = n_tiles workgroups.
using G1 = Geo<CONV_FH, CONV_FW, CONV_BX, CONV_BY, CONV_TX, CONV_TY, CONV_USE_LDS, CONV_UNROLL, CONV_VIN, CONV_VOUT>;
extern "C" __global__ void __launch_bounds__(G1::NT) CONV_WAVES
CONV_NAME(const float* __restrict__ in, const float* __restrict__ filt,
          float* __restrict__ out, int H, int W, int tiles_x, int n_tiles, u32 in_bytes)
{
    __shared__ __attribute__((aligned(16))) float lds[G1::LDS_FLOATS];
    const int t = xcd_remap((int)blockIdx.x, n_tiles);
    const int tile_y = t / tiles_x;
    const int tile_x = t - tile_y * tiles_x;
    conv_tile<CONV_FH, CONV_FW, CONV_BX, CONV_BY, CONV_TX, CONV_TY, CONV_USE_LDS, CONV_UNROLL, CONV_VIN, CONV_VOUT>(
        in, filt, out, H, W, in_bytes, tile_x, tile_y, lds);
}
#else
#if CONV_FCONST
#error "the batched kernel reads each problem's own filter through its pointer"
#endif
// One problem of a batch, as the host library lays it out in device memory.
struct ConvDesc {
    const float* in;
    const float* filt;
    float* out;
    int H, W;
    int tiles_x;
    int tile_begin;   // first tile of this problem in the tile list
    u32 in_bytes;
    int n_tiles;      // tiles of this problem
};

// The descriptor of tile t, in scalar registers (it is the same for every
// lane, and all addressing and the filter taps follow from it). There is no
// 16-bit scalar load on gfx9: the aligned dword that holds the tile's owner is
// read (the library allocates its tables in whole dwords). The descriptor comes
// in one go, so what a workgroup waits for before its first input load is
// arguments, owner, descriptor, one after another. With a vector load for the
// owner, the descriptor field by field, and its pointers read through as if
// they could point anywhere (see TapPtr), one image of 4096 x 4096 took 5 x 5
// 23.9 us (now 21.3), 9 x 9 43.1 (41.1) and 3 x 3 21.4 (20.0), and 64 images up
// to 2048 took 225 us (214).
static __device__ __forceinline__ ConvDesc tile_desc(const ConvDesc* __restrict__ descs,
                                                     const unsigned short* __restrict__ owner, int t)
{
#if defined(__AMDGCN__)
    typedef const __attribute__((address_space(4))) u32 cu32;
    typedef const __attribute__((address_space(4))) u32x4 cu32x4;
    struct Words {
        u32x4 a, b, c;
    };
    const unsigned long long at = (unsigned long long)(owner + t);
    const u32 who = (*(cu32*)(at & ~3ull) >> ((u32)(at & 2u) * 8u)) & 0xffffu;
    cu32x4* from = (cu32x4*)(unsigned long long)(descs + who);
    const Words w = {from[0], from[1], from[2]};
    return __builtin_bit_cast(ConvDesc, w);
#else
    return descs[owner[t]];
#endif
}

// Many images with the same filter size: a grid of at least 8 workgroups
// walks the group's tile list (the library launches one workgroup per tile;
// a smaller grid gives each workgroup several). The tiles of XCD x (=
// workgroup id mod 8) form one contiguous range, shared out by stride among
// that XCD's workgroups; owner[t] names the problem of tile t.
using G1 = Geo<CONV_FH, CONV_FW, CONV_BX, CONV_BY, CONV_TX, CONV_TY, CONV_USE_LDS, CONV_UNROLL, CONV_VIN, CONV_VOUT>;
extern "C" __global__ void __launch_bounds__(G1::NT) CONV_WAVES
CONV_NAME(const ConvDesc* __restrict__ descs, const unsigned short* __restrict__ owner, int total_tiles)
{
    __shared__ __attribute__((aligned(16))) float lds[G1::LDS_FLOATS];
    const int G = (int)gridDim.x;
#if defined(__AMDGCN__)
    // The arguments are fetched together, not each where it is first used.
    asm volatile("" : : "s"(descs), "s"(owner), "s"(total_tiles), "s"(G));
#endif
    const int xcd = (int)blockIdx.x & 7;
    const int first = (int)blockIdx.x >> 3;
    const int stride = (G - xcd + 7) >> 3;
    const int q = total_tiles >> 3, rem = total_tiles & 7;
    const int begin = xcd * q + min_(xcd, rem);
    const int count = q + (xcd < rem ? 1 : 0);
    for (int k = first; k < count; k += stride) {
        const int t = begin + k;
        const ConvDesc d = tile_desc(descs, owner, t);
        const int lt = t - d.tile_begin;
        if ((unsigned)lt >= (unsigned)d.n_tiles)
            continue;  // inconsistent tables: skip rather than store out of range (uniform)
        const int tile_y = lt / d.tiles_x;
        const int tile_x = lt - tile_y * d.tiles_x;
        if (CONV_USE_LDS && k != first)
            __syncthreads();  // every thread is done with the previous tile's LDS
        conv_tile<CONV_FH, CONV_FW, CONV_BX, CONV_BY, CONV_TX, CONV_TY, CONV_USE_LDS, CONV_UNROLL, CONV_VIN, CONV_VOUT>(
            d.in, d.filt, d.out, d.H, d.W, d.in_bytes, tile_x, tile_y, lds);
    }
}
#endif
