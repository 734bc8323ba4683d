// Projections of a decoder layer: C[M,N] = A[M,K] * W[N,K]^T with bf16 inputs, fp32 accumulation on
// the matrix cores, and three epilogues: plain, + residual, SwiGLU.
//
// Both operands are K-contiguous, so a lane's MFMA operand (8 consecutive k of one row / column)
// is one 16-byte LDS read.  Four kernels share the work: gemm_big_kernel (prefill-sized problems: 256x256
// tiles, operands global -> LDS by DMA into a five-slot ring), gemm_mid_kernel (65 to 2048 rows: tiles sized to the
// batch), both of 16x16x32 products, gemm_skinny_kernel (up to 64 rows: the weights are streamed once, split over K) and
// gemm_kernel below (everything else: K tails, odd widths, no workspace), both of 32x32x16 products.  gemm_kernel
// stages tiles global -> registers -> LDS, double buffered, one barrier per 64-wide K step, LDS rows padded by 16 bytes
// so that the operand reads of 16 consecutive rows fall in distinct banks.
#include <type_traits>

#include "common.h"

namespace bz {

#ifndef BZ_FP32_DEBUG

constexpr int kBK = 64;            // K step per LDS stage
constexpr int kLdsRow = kBK + 8;   // padded row length in elements (144 bytes)

template <int BM, int BN>
constexpr int gemm_lds_bytes() { return 2 * (BM + BN) * kLdsRow * (int)sizeof(bf16); }

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of logical tile
// ids so tiles that share operand rows meet in one L2.
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    const int xcd = bid & 7, local = bid >> 3;
    const int base = nb >> 3, rem = nb & 7;
    return xcd * base + (xcd < rem ? xcd : rem) + local;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int MODE>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void gemm_kernel(const bf16* __restrict__ A,
                                                                      const bf16* __restrict__ W,
                                                                      const bf16* R, bf16* C, int M, int N,
                                                                      int K, int tiles_m, int tiles_n) {
    constexpr int THREADS = WAVES_M * WAVES_N * 64;
    constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
    constexpr int MI = WTM / 32, NJ = WTN / 32;
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be a multiple of the MFMA block");
    static_assert(MODE != 2 || NJ % 2 == 0, "SwiGLU needs gate and up blocks in the same wave");
    constexpr int ROWS_PER_PASS = THREADS / 8;      // 8 vectors of 8 elements per 64-wide row
    constexpr int PA = BM / ROWS_PER_PASS, PB = BN / ROWS_PER_PASS;
    static_assert(BM % ROWS_PER_PASS == 0 && BN % ROWS_PER_PASS == 0, "tile rows vs loader passes");
    constexpr int OUT_BN = (MODE == 2) ? BN / 2 : BN;   // output columns per tile

    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16* As = reinterpret_cast<bf16*>(smem_raw);                 // [2][BM][kLdsRow]
    bf16* Bs = As + 2 * BM * kLdsRow;                             // [2][BN][kLdsRow]

    // ---- tile coordinates (grouped along M for L2 reuse of the weight tile) ----
    const int pid = xcd_remap(blockIdx.x, tiles_m * tiles_n);
    constexpr int GROUP = 8;
    const int width = GROUP * tiles_n;
    const int group_id = pid / width;
    const int first_m = group_id * GROUP;
    const int gsize = (tiles_m - first_m < GROUP) ? (tiles_m - first_m) : GROUP;
    const int tile_m = first_m + (pid % width) % gsize;
    const int tile_n = (pid % width) / gsize;
    const int m0 = tile_m * BM;
    const int n0 = tile_n * OUT_BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int lrow = lane & 31, lk = lane >> 5;

    // ---- loader mapping ----
    const int vcol = tid & 7;             // which 8-element vector of the 64-wide row
    const int vrow = tid >> 3;            // row within a pass
    const bf16* a_ptr[PA];
    const bf16* b_ptr[PB];
#pragma unroll
    for (int p = 0; p < PA; ++p) {
        int r = m0 + vrow + p * ROWS_PER_PASS;
        if (r > M - 1) r = M - 1;
        a_ptr[p] = A + (size_t)r * K + vcol * 8;
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        const int lr = vrow + p * ROWS_PER_PASS;      // row in the LDS B tile
        int r;
        if (MODE == 2) {
            const bool up = lr >= BN / 2;
            int f = n0 + (up ? lr - BN / 2 : lr);
            if (f > N - 1) f = N - 1;
            r = up ? N + f : f;
        } else {
            r = n0 + lr;
            if (r > N - 1) r = N - 1;
        }
        b_ptr[p] = W + (size_t)r * K + vcol * 8;
    }

    uint4 ra[PA], rb[PB];
    auto load_tile = [&](int k0) {
        const bool kin = (k0 + vcol * 8) < K;
#pragma unroll
        for (int p = 0; p < PA; ++p)
            ra[p] = kin ? *reinterpret_cast<const uint4*>(a_ptr[p] + k0) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int p = 0; p < PB; ++p)
            rb[p] = kin ? *reinterpret_cast<const uint4*>(b_ptr[p] + k0) : make_uint4(0, 0, 0, 0);
    };
    auto store_tile = [&](int buf) {
        bf16* as = As + buf * BM * kLdsRow;
        bf16* bs = Bs + buf * BN * kLdsRow;
#pragma unroll
        for (int p = 0; p < PA; ++p)
            *reinterpret_cast<uint4*>(as + (vrow + p * ROWS_PER_PASS) * kLdsRow + vcol * 8) = ra[p];
#pragma unroll
        for (int p = 0; p < PB; ++p)
            *reinterpret_cast<uint4*>(bs + (vrow + p * ROWS_PER_PASS) * kLdsRow + vcol * 8) = rb[p];
    };

    f32x16 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // LDS row of the wave's j-th column block
    int brow[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (MODE == 2) {
            constexpr int HJ = NJ / 2 > 0 ? NJ / 2 : 1;
            const bool up = j >= HJ;
            const int jj = up ? j - HJ : j;
            brow[j] = (up ? BN / 2 : 0) + (wn * HJ + jj) * 32 + lrow;
        } else {
            brow[j] = (wn * NJ + j) * 32 + lrow;
        }
    }

    const int nk = (K + kBK - 1) / kBK;
    load_tile(0);
    store_tile(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) load_tile((kt + 1) * kBK);
        const bf16* as = As + cur * BM * kLdsRow;
        const bf16* bs = Bs + cur * BN * kLdsRow;
#pragma unroll
        for (int ks = 0; ks < kBK / 16; ++ks) {
            bf16x8 af[MI], bfr[NJ];
#pragma unroll
            for (int i = 0; i < MI; ++i)
                af[i] = *reinterpret_cast<const bf16x8*>(as + (wm * WTM + i * 32 + lrow) * kLdsRow + ks * 16 + lk * 8);
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                bfr[j] = *reinterpret_cast<const bf16x8*>(bs + brow[j] * kLdsRow + ks * 16 + lk * 8);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) store_tile(cur ^ 1);
        __syncthreads();
    }

    // ---- epilogue: lane holds column (lane%32) and rows 8*(r/4) + 4*(lane/32) + r%4 of each block
    if (MODE == 2) {
        constexpr int HJ = NJ / 2 > 0 ? NJ / 2 : 1;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < HJ; ++j) {
                const int col = n0 + (wn * HJ + j) * 32 + lrow;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = m0 + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * lk + (r & 3);
                    if (row < M && col < N) {
                        const float g = acc[i][j][r], u = acc[i][j + HJ][r];
                        const float sg = silu_fast(g);
                        C[(size_t)row * N + col] = (bf16)(sg * u);
                    }
                }
            }
    } else {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int col = n0 + (wn * NJ + j) * 32 + lrow;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = m0 + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * lk + (r & 3);
                    if (row < M && col < N) {
                        float v = acc[i][j][r];
                        if (MODE == 1) v += (float)R[(size_t)row * N + col];
                        C[(size_t)row * N + col] = (bf16)v;
                    }
                }
            }
    }
}

// ---------------------------------------------------------------------------------------------
// Large-tile kernel for prefill-sized problems (K a multiple of 64, N a multiple of 4):
// 256x256x64 workgroup tile, 4 waves, 128x128 per wave (256 accumulator registers).  Operands reach
// LDS by direct global->LDS loads (16 bytes per lane, no register staging).  A wave's load
// instruction writes 1 KiB of LDS in lane order, i.e. 8 rows of 128 bytes; bank conflicts are
// avoided by permuting WHICH 16-byte piece of its row each lane fetches (an XOR swizzle applied on
// the global side) and reading operands with the same permutation.  The weight tile feeds the
// MFMA's row operand and the activation tile its column operand, so a lane ends up with runs of
// consecutive output features of one token (8 with the row order described at big_row_feature:
// 16-byte stores), and gate/up of the same feature in the same lane for the SwiGLU epilogue.
//
// With real operand values the chip holds the matrix pipes back for power, not for issue: a loop of nothing but
// MFMAs on random data sustains 1.79 PFLOP/s with the 32x32x16 form and 2.05 with the 16x16x32 form (2.44 and
// 2.42 on zeros), because the 16x16x32 form touches its accumulators half as often per product.  So the tile is
// built of 16x16x32 products, 8 x 8 blocks of four accumulators per wave.  Against the same kernel built of 32x32x16
// products (same tile, ring and loads), microseconds: 8192 rows, 8192 -> gate/up 28672 5326 -> 4943 (1.45 -> 1.56
// PFLOP/s), down 2735 -> 2518, qkv 10240 963 -> 888; 4973 rows, 4096 -> gate/up 11008 663 -> 616, qkv 12288 383 -> 349.
//
// LDS is a ring of five 32 KiB slots, each holding one operand's 256 rows of one k-tile: the tile
// being multiplied, the next one, and the activation half of the one after.  What decides the
// schedule is the cost of ISSUING a load: a 1 KiB load holds its wave's instruction stream for
// about 64 cycles when the four waves issue together (the address unit is shared), and a wave that
// cannot issue cannot feed the matrix pipe either.  So loads go out one every few MFMAs, spread
// over the whole tile, into the two slots the previous tile released, and the wait before a
// tile's barrier leaves the newest 32 KiB in flight.
// ---------------------------------------------------------------------------------------------
constexpr int kBigSlot = 256 * kBK * (int)sizeof(bf16);      // 32768: one operand's 256 rows of one k-tile
constexpr int kBigSlots = 5;

__device__ __forceinline__ int swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// Which feature sits where.  A 16x16x32 MFMA leaves lane group h (lanes 16h .. 16h+15) of the output with rows
// 4h .. 4h+3 of the row operand.  The weight rows of a 32-feature block pair are therefore laid into LDS in a permuted
// order - row 4h + e of block b (b = 0, 1) holds feature 8h + 4b + e - so that a lane's four registers of block 0 and
// four of block 1 are the 8 consecutive features 8h .. 8h+7 of one token: 16-byte output stores, 64 contiguous bytes
// per token and instruction.  The permutation costs nothing: it only changes which global row a loader lane fetches.
__device__ __forceinline__ int big_row_feature(int rho) {            // row inside a block pair -> feature inside it
    const int b = rho >> 4, h = (rho >> 2) & 3, e = rho & 3;
    return 8 * h + 4 * b + e;
}

// acc += w * x, one 16x16x32 product, accumulating in place.  Written out because the compiler, given 64 accumulators
// that fill all 256 accumulation registers, takes the form with a separate destination and rotates the accumulators
// through copies (196 register moves and 97 waits per k-tile).  The compiler still counts the LDS reads behind the
// operands; what it no longer sees is the time until a result may be read by other instructions: mfma16_settle().
__device__ __forceinline__ void mfma16(f32x4& acc, const bf16x8& w, const bf16x8& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}
// The same at the end of a k-tile: behind the last one (left == 1) follow sixteen wait states, of which a 4-pass product
// needs at most 11 before its result may be read.  They are part of the product's own statement and inside the loop,
// because nothing else holds the register allocator back: with a separate wait behind the loop it placed its copies of
// the accumulators between the last product and the wait.
__device__ __forceinline__ void mfma16_settle(f32x4& acc, const bf16x8& w, const bf16x8& x, int left) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\t"
                 "s_cmp_lg_u32 %3, 1\n\t"
                 "s_cbranch_scc1 1\n\t"          // over the next instruction
                 "s_nop 15"
                 : "+a"(acc) : "v"(w), "v"(x), "s"(left) : "scc");
}

// logical tile id -> tile coordinates: groups of 4 tile rows, walked column by column, so that the
// tiles running together on an XCD share operand rows in its L2
struct BigTile { int m0, n0; };
template <int MODE>
__device__ __forceinline__ BigTile big_tile_of(int pid, int tiles_m, int tiles_n) {
    constexpr int OUT_BN = (MODE == 2) ? 128 : 256;
    constexpr int GROUP = 4;
    const int width = GROUP * tiles_n;
    const int group_id = pid / width;
    const int first_m = group_id * GROUP;
    const int gsize = (tiles_m - first_m < GROUP) ? (tiles_m - first_m) : GROUP;
    const int tile_m = first_m + (pid % width) % gsize;
    const int tile_n = (pid % width) / gsize;
    return BigTile{tile_m * 256, tile_n * OUT_BN};
}

// First output feature, inside the tile, of a wave's feature pair p (32 features; SwiGLU: of both factors).
template <int MODE>
__device__ __forceinline__ int big_pair_feature(int wn, int p) { return wn * (MODE == 2 ? 64 : 128) + p * 32; }

// 8 consecutive output features n .. n+7 of one token: one 16-byte access when rows are multiples of 8 features,
// else (N % 4 == 0) two of 8 bytes, each behind its own bound.
__device__ __forceinline__ void big_store8(bf16* crow, int n, int N, const float (&o)[8]) {
    bf16x8 w;
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = (bf16)o[e];
    if ((N & 7) == 0) {
        if (n < N) *reinterpret_cast<bf16x8*>(crow + n) = w;
    } else {
        if (n < N) *reinterpret_cast<bf16x4*>(crow + n) = __builtin_shufflevector(w, w, 0, 1, 2, 3);
        if (n + 4 < N) *reinterpret_cast<bf16x4*>(crow + n + 4) = __builtin_shufflevector(w, w, 4, 5, 6, 7);
    }
}
// the same features of the residual; past the end a valid address is read and its value never used
__device__ __forceinline__ bf16x8 big_load8(const bf16* rrow, int n, int N) {
    if ((N & 7) == 0) return *reinterpret_cast<const bf16x8*>(rrow + (n > N - 8 ? N - 8 : n));
    const bf16x4 lo = *reinterpret_cast<const bf16x4*>(rrow + (n > N - 4 ? N - 4 : n));
    const bf16x4 hi = *reinterpret_cast<const bf16x4*>(rrow + (n + 4 > N - 4 ? N - 4 : n + 4));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Tile scheduling.  A launch runs one workgroup per CU at a time, so `tiles` whole tiles take
// ceil(tiles / 256) rounds and a last round with few tiles wastes most of the chip.  The first
// n_dp tiles (a multiple of 256) are computed whole by one launch; each of the remaining tiles is
// cut into `splits` ranges of K, one workgroup each (a second launch of the PARTIAL instantiation,
// which starts as the first drains), which write fp32 partial tiles to `ws`; a small third kernel
// adds the partial tiles in range order and applies the epilogue.  The cut is a function of the
// problem shape only.
template <int MODE, bool PARTIAL>
__global__ __launch_bounds__(256, 1) void gemm_big_kernel(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                           const bf16* R, bf16* C, int M, int N, int K,
                                                           int tiles_m, int tiles_n, int n_dp, int splits,
                                                           float* __restrict__ ws) {
    constexpr int NCH = 8;                     // 1 KiB chunks of each tile filled by one wave
    constexpr int NB = 8;                      // 16-wide blocks of a wave's 128 features / tokens
    constexpr int NMMA = NB * NB;              // MFMAs per k-step of 32
    constexpr int NFETCH = 2 * NB;             // LDS operand reads per k-step
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];

    const int nk = K / kBK;
    int pid, kt0 = 0, kt1 = nk;
    const int slot = blockIdx.x;                       // PARTIAL: (split tile, K range)
    if (!PARTIAL) {
        pid = xcd_remap(blockIdx.x, n_dp);
    } else {
        pid = n_dp + slot / splits;
        const int per = (nk + splits - 1) / splits;
        kt0 = (slot % splits) * per;
        kt1 = (kt0 + per < nk) ? kt0 + per : nk;
    }
    const BigTile bt = big_tile_of<MODE>(pid, tiles_m, tiles_n);
    const int m0 = bt.m0, n0 = bt.n0;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane & 15, lg = lane >> 4;

    // ---- loader: this wave fills chunks q = wave*NCH + j (rows 8q .. 8q+7) of both tiles.  Addresses
    // are a uniform base (advanced per K tile) plus a per-lane 32-bit byte offset.
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    uint32_t a_off[NCH], b_off[NCH];
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        const int row = (wave * NCH + j) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ swz(row);
        int ar = m0 + row;
        if (ar > M - 1) ar = M - 1;
        a_off[j] = ((uint32_t)ar * (uint32_t)K + c * 8) * 2u;
        const int frow = (row & ~31) | big_row_feature(row & 31);     // the feature this LDS row holds
        int br;
        if (MODE == 2) {
            const bool up = frow >= 128;
            int f = n0 + (up ? frow - 128 : frow);
            if (f > N - 1) f = N - 1;
            br = up ? N + f : f;
        } else {
            br = n0 + frow;
            if (br > N - 1) br = N - 1;
        }
        b_off[j] = ((uint32_t)br * (uint32_t)K + c * 8) * 2u;
    }
    // Unit u = 2t is the activation half of k-tile t, u = 2t + 1 its weight half; unit u lives in slot
    // u % 5.  Piece q in [0, NCH) of a unit is this wave's q-th 1 KiB chunk.  Past the last k-tile the
    // last one is fetched again (into a slot nobody reads any more) so that every tile issues the
    // same number of loads and the wait counts below hold for every tile.
    // Loads take the buffer form: resource in scalar registers, the lane's byte offset in one vector register,
    // the k-tile's byte offset in a scalar register.  The flat form made the compiler add a 64-bit base to the
    // offset with a vector instruction before every load, and vector ALU instructions in this loop cost matrix
    // time (16 of them per k-tile and wave: 1.3 - 1.5 % of the GEMM).
    const __amdgpu_buffer_rsrc_t rsrc_a =
        __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)((uint32_t)M * (uint32_t)K * 2u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(
        (void*)W, 0, (int)((uint32_t)(MODE == 2 ? 2 * N : N) * (uint32_t)K * 2u), 0x00020000);
    auto issue_piece = [&](int kt, int slot, bool weights, int q) {
        unsigned char* sa = smem_raw + slot * kBigSlot + (wave_u * NCH + q) * 1024;
        const int t = kt < kt1 ? kt : kt1 - 1;
        if (!weights) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lptr_t)sa, 16, (int)a_off[q], t * (kBK * 2), 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w, (lptr_t)sa, 16, (int)b_off[q], t * (kBK * 2), 0, 0);
    };
    auto issue_unit = [&](int kt, int slot, bool weights) {
#pragma unroll
        for (int q = 0; q < NCH; ++q) issue_piece(kt, slot, weights, q);
    };

    f32x4 acc[NB][NB];      // [feature block][token block]
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][i][r] = 0.f;

    // ---- operand addresses inside a slot: per-lane part in one register per k-step and operand, the 16-row blocks
    // being immediate offsets from it (block j of the weights: 16j rows on; SwiGLU: blocks 4..7 are the up factor,
    // 128 rows further)
    int xk[2], wk[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int piece = ((ks * 4 + lg) ^ swz(lrow)) * 16;
        xk[ks] = (wm * 128 + lrow) * 128 + piece;
        wk[ks] = (wn * (MODE == 2 ? 64 : 128) + lrow) * 128 + piece;
    }
    constexpr int kBlk = 16 * 128;
    auto w_blk = [](int j) { return (MODE == 2 && j >= NB / 2) ? 128 * 128 + (j - NB / 2) * kBlk : j * kBlk; };

    // ---- main loop.  Every k-step is NMMA MFMAs in a fixed order; between them, one by one, go the LDS reads that
    // fetch the operands of the NEXT k-step (behind every second MFMA of the first half) and the global->LDS loads
    // (behind every eighth MFMA, one that has no LDS read behind it).  The order is pinned with scheduling barriers so
    // the matrix pipe never waits behind a burst of memory instructions.  Other spacings (reads every third MFMA, loads
    // in the second half only, the four waves' loads a few MFMAs apart) measure within 1 % of this one: the loop is
    // bound by power, not by issue.  On random data, 8192x8192 into gate/up of 28672, a tile's k-step stream without its
    // global->LDS loads runs 15 % faster, without its LDS reads 9 %, without both at the rate of bare MFMAs; with every
    // load hitting the L2 6 %.  The tile barrier sits before the second k-step, whose operands are already in
    // registers; it is a bare s_barrier (the waits are written out here; a full __syncthreads would drain the loads
    // that are meant to stay in flight).
    //
    // The two slots tile i - 1 released at its barrier are refilled as follows: second k-step of tile i - 1: weights
    // of tile i + 1 (needed first); first k-step of tile i: activations of tile i + 2.  Before the barrier of tile i
    // everything but those activations must have landed.
    bf16x8 xf[2][NB], wf[2][NB];
    auto fetch_piece = [&](const unsigned char* sx, const unsigned char* sw_, int ks, int buf, int q) {   // order of first use
        if (q == 0) wf[buf][0] = *reinterpret_cast<const bf16x8*>(sw_ + wk[ks]);
        else if (q <= NB) xf[buf][q - 1] = *reinterpret_cast<const bf16x8*>(sx + xk[ks] + (q - 1) * kBlk);
        else wf[buf][q - NB] = *reinterpret_cast<const bf16x8*>(sw_ + wk[ks] + w_blk(q - NB));
    };
    // one k-step: MFMAs from buffer `cur`; fetch k-step `nks` of the tile in slots (sx, sw_) into the
    // other buffer; request the NCH pieces of one operand of k-tile `ikt` into slot `islot`; `left`: k-tiles from this
    // one on (the second k-step ends them)
    auto kstep = [&](int cur, const unsigned char* sx, const unsigned char* sw_, int nks, int ikt, int islot, bool iweights,
                     int left) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < NMMA; ++q) {
            const int j = q >> 3, i = q & 7;
            if (cur == 1 && q == NMMA - 1) mfma16_settle(acc[j][i], wf[cur][j], xf[cur][i], left);
            else mfma16(acc[j][i], wf[cur][j], xf[cur][i]);
            if (q % 2 == 0 && q / 2 < NFETCH) fetch_piece(sx, sw_, nks, cur ^ 1, q / 2);
            if (q % 8 == 5) issue_piece(ikt, islot, iweights, q / 8);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    if (M > 0x7fffffff / K || 2 * N > 0x7fffffff / K) return;    // 32-bit offsets (checked on the host too)
    const int n = kt1 - kt0;                           // k-tiles of this workgroup, >= 1
    issue_unit(kt0, 0, false);
    issue_unit(kt0, 1, true);
    issue_unit(kt0 + 1, 2, false);
    issue_unit(kt0 + 1, 3, true);
    __builtin_amdgcn_s_waitcnt(0x4F70);                // vmcnt(16): tile kt0 landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < NFETCH; ++q) fetch_piece(smem_raw, smem_raw + kBigSlot, 0, 0, q);
    int sa = 0;                                        // slot of the current tile's activations; its weights follow
    for (int i = 0; i < n; ++i) {
        const int sw1 = (sa + 1 >= kBigSlots) ? sa + 1 - kBigSlots : sa + 1;
        const int na = (sa + 2 >= kBigSlots) ? sa + 2 - kBigSlots : sa + 2;      // next tile's slots
        const int nw = (sa + 3 >= kBigSlots) ? sa + 3 - kBigSlots : sa + 3;
        const int fa2 = (sa + 4 >= kBigSlots) ? sa + 4 - kBigSlots : sa + 4;     // where tile i + 2's activations go
        kstep(0, smem_raw + sa * kBigSlot, smem_raw + sw1 * kBigSlot, 1, kt0 + i + 2, fa2, false, n - i);
        // tile i + 1 has landed (only the NCH newest loads, activations of tile i + 2, may be in flight);
        // own LDS reads of tile i are done
        __builtin_amdgcn_s_waitcnt(0x0078);            // vmcnt(8) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        // tile i + 2's weights into the slot this tile's activations just left
        kstep(1, smem_raw + na * kBigSlot, smem_raw + nw * kBigSlot, 0, kt0 + i + 2, sa, true, n - i);
        sa = na;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                // no LDS write may be in flight when the workgroup ends

    if (PARTIAL) {
        // partial tile in accumulator order: every (wave, j, i) is 1 KiB of `ws`, four values per lane
        float* base = ws + (size_t)slot * 65536 + (size_t)wave_u * (NB * NB * 256) + lane * 4;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            // a 16-token block wholly past the last row is never read back (a few hundred rows fill
            // only part of a 256-row tile, and the partial tiles are most of the traffic then)
            if (m0 + (wave_u >> 1) * 128 + i * 16 < M) {
#pragma unroll
                for (int j = 0; j < NB; ++j) *reinterpret_cast<f32x4*>(base + (j * NB + i) * 256) = acc[j][i];
            }
            __builtin_amdgcn_sched_barrier(0);         // one block at a time: few registers besides the accumulators are free
        }
        return;
    }
    constexpr int NP = (MODE == 2) ? 2 : 4;            // feature pairs a wave writes
    // R may be C itself (the residual stream is updated in place); a lane reads exactly the addresses it
    // writes, so a token block's residual values are fetched together, and the next block's before this
    // block's stores go out (written as load-then-store the loads would queue behind the stores).
    bf16x8 rv[2][NP];
    auto load_r = [&](int i, int buf) {
        int m = m0 + wm * 128 + i * 16 + lrow;
        if (m > M - 1) m = M - 1;                       // rows past the end: a valid address, value unused
#pragma unroll
        for (int p = 0; p < NP; ++p)
            rv[buf][p] = big_load8(R + (size_t)m * N, n0 + big_pair_feature<MODE>(wn, p) + 8 * lg, N);
    };
    if (MODE == 1) load_r(0, 0);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (MODE == 1 && i + 1 < NB) load_r(i + 1, (i + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        const int m = m0 + wm * 128 + i * 16 + lrow;
        if (m < M) {
            bf16* crow = C + (size_t)m * N;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                float o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = acc[2 * p + (e >> 2)][i][e & 3];
                    if (MODE == 2) o[e] = silu_fast(v) * acc[NB / 2 + 2 * p + (e >> 2)][i][e & 3];
                    else if (MODE == 1) o[e] = v + (float)rv[i & 1][p][e];
                    else o[e] = v;
                }
                big_store8(crow, n0 + big_pair_feature<MODE>(wn, p) + 8 * lg, N, o);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Adds the partial tiles of one split tile in range order and applies the epilogue.  One wave per (wave of the
// main kernel, feature pair p, token block i): a lane sums the 8 values behind one token's 8 consecutive features.
// The ranges are taken four at a time, then two, then one, every batch's loads going out together; the sums run in
// range order whatever the batching.  Grid (split tiles, units / 4).
template <int MODE>
__global__ __launch_bounds__(256) void gemm_big_fixup(const float* __restrict__ ws, const bf16* R, bf16* C, int M,
                                                      int N, int tiles_m, int tiles_n, int n_dp, int splits) {
    constexpr int NB = 8;
    constexpr int NP = (MODE == 2) ? 2 : 4;             // feature pairs per wave of the main kernel
    constexpr int NV = (MODE == 2) ? 2 : 1;             // factors behind one output
    const int tile = blockIdx.x;
    const BigTile bt = big_tile_of<MODE>(n_dp + tile, tiles_m, tiles_n);
    const int lane = threadIdx.x & 63;
    const int u = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int i = u & 7, p = (u >> 3) % NP, wave = (u >> 3) / NP;
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane & 15, lg = lane >> 4;
    if (bt.m0 + wm * 128 + i * 16 >= M) return;          // block past the last row: nothing was stored for it
    const int m = bt.m0 + wm * 128 + i * 16 + lrow;
    const int n = bt.n0 + big_pair_feature<MODE>(wn, p) + 8 * lg;
    // the residual does not depend on the sums: requested first
    bf16x8 rv;
    if (MODE == 1) rv = big_load8(R + (size_t)(m < M ? m : M - 1) * N, n, N);
    f32x4 acc[NV][2];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[v][b][e] = 0.f;
    const float* base = ws + (size_t)tile * splits * 65536 + (size_t)wave * (NB * NB * 256) + lane * 4;
    auto batch = [&](int s0, auto nb) {
        constexpr int NS = decltype(nb)::value;
        f32x4 t[NS][NV][2];
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    t[q][v][b] = *reinterpret_cast<const f32x4*>(base + (size_t)(s0 + q) * 65536 +
                                                                 ((v * (NB / 2) + 2 * p + b) * NB + i) * 256);
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[v][b][e] += t[q][v][b][e];
    };
    int s0 = 0;
    for (; s0 + 4 <= splits; s0 += 4) batch(s0, std::integral_constant<int, 4>());
    if (s0 + 2 <= splits) { batch(s0, std::integral_constant<int, 2>()); s0 += 2; }
    if (s0 < splits) batch(s0, std::integral_constant<int, 1>());
    if (m >= M) return;
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = acc[0][e >> 2][e & 3];
        if (MODE == 2) o[e] = silu_fast(v) * acc[NV - 1][e >> 2][e & 3];
        else if (MODE == 1) o[e] = v + (float)rv[e];
        else o[e] = v;
    }
    big_store8(C + (size_t)m * N, n, N, o);
}

struct BigPlan {
    int tiles_m, tiles_n, n_dp, tail, splits;
    size_t ws_bytes;
};

static BigPlan big_plan(int mode, int M, int N, int K) {
    BigPlan p;
    const int out_bn = (mode == 2) ? 128 : 256;
    p.tiles_m = (M + 255) / 256;
    p.tiles_n = (N + out_bn - 1) / out_bn;
    const int tiles = p.tiles_m * p.tiles_n, nk = K / kBK;
    constexpr int kCUs = 256, kMaxTail = 128, kMaxSplits = 16, kMinKt = 4;
    p.n_dp = tiles;
    p.tail = 0;
    p.splits = 1;
    p.ws_bytes = 0;
    const int full = tiles / kCUs * kCUs, rest = tiles - full;
    // rest <= kMaxTail: the last round is at most half full (then two ranges of K per tile fit the chip).
    // full == 0: fewer tiles than CUs altogether; every tile is split, whatever their number, so that the whole chip
    // streams the weights.
    if (rest > 0 && (rest <= kMaxTail || full == 0)) {
        int sp = kCUs / rest;
        if (sp > kMaxSplits) sp = kMaxSplits;
        if (sp > nk / kMinKt) sp = nk / kMinKt;
        if (sp >= 2) {
            const int per = (nk + sp - 1) / sp;
            sp = (nk + per - 1) / per;               // every range non-empty
            p.n_dp = full;
            p.tail = rest;
            p.splits = sp;
            p.ws_bytes = (size_t)rest * sp * 65536 * sizeof(float);
        }
    }
    return p;
}

static bool big_ok(int M, int N, int K) {
    return M > 64 && K % kBK == 0 && N % 4 == 0 && (uint64_t)M * K < 0x7fffffffull &&
           (uint64_t)2 * N * K < 0x7fffffffull;          // the large-tile kernel uses 32-bit byte offsets / 2
}

// The large-tile kernel needs the CU's whole 160 KiB of LDS; if the runtime does not grant it (asked once per
// instantiation and device) the caller takes the 128x128 kernel instead.
template <int MODE>
static bool big_available() {
    constexpr int LDS = kBigSlots * kBigSlot;
    static LdsLimit whole, partial;
    const bool a = whole.raise(reinterpret_cast<const void*>(gemm_big_kernel<MODE, false>), LDS);
    const bool b = partial.raise(reinterpret_cast<const void*>(gemm_big_kernel<MODE, true>), LDS);
    return a && b;
}

template <int MODE>
static void launch_big(const bf16* a, const bf16* w, const bf16* r, bf16* c, int M, int N, int K, float* ws,
                       size_t ws_bytes, hipStream_t st) {
    constexpr int LDS = kBigSlots * kBigSlot;
    auto kern = gemm_big_kernel<MODE, false>;
    auto kern_part = gemm_big_kernel<MODE, true>;
    BigPlan p = big_plan(MODE, M, N, K);
    if (p.tail > 0 && (ws == nullptr || ws_bytes < p.ws_bytes)) {     // no scratch: every tile whole
        p.n_dp = p.tiles_m * p.tiles_n;
        p.tail = 0;
        p.splits = 1;
    }
    if (p.n_dp > 0)
        hipLaunchKernelGGL(kern, dim3(p.n_dp), dim3(256), LDS, st, a, w, r, c, M, N, K, p.tiles_m, p.tiles_n,
                           p.n_dp, p.splits, ws);
    if (p.tail > 0) {
        hipLaunchKernelGGL(kern_part, dim3(p.tail * p.splits), dim3(256), LDS, st, a, w, r, c, M, N, K,
                           p.tiles_m, p.tiles_n, p.n_dp, p.splits, ws);
        constexpr int kUnits = 4 * ((MODE == 2) ? 2 : 4) * 8;           // waves * feature pairs * token blocks
        hipLaunchKernelGGL(gemm_big_fixup<MODE>, dim3(p.tail, kUnits / 4), dim3(256), 0, st, ws, r, c, M, N, p.tiles_m,
                           p.tiles_n, p.n_dp, p.splits);
    }
}

// ---------------------------------------------------------------------------------------------
// Mid-sized kernel: 65 to 2048 rows (K a multiple of 64, N of 4).  The decode kernel would re-read the weights once
// per 64 rows, and of 256x256 tiles half would be padding and fewer exist than CUs.  The tile is BM tokens x BN weight
// rows, both chosen by mid_plan so that the padded problem is one round (or a few full ones) of workgroups, over one
// or several ranges of K.  Four waves, WT of them along the tokens; a wave multiplies NBT x NBF blocks of 16x16x32.
//
// What bounds it is the delivery of the operands into LDS: a workgroup moves (BM + BN) * 128 bytes per k-tile at 57
// bytes per ns and CU (13 TB/s over the chip, weights from HBM, activations from L2).  Leaving the MFMAs out changes
// nothing (7B gate/up at 301 rows: 59.0 -> 59.4 us), and neither do four more waves that do nothing but request; with both
// operands served by the L2 it takes 44 us.  So tiles are as square as filling the chip allows.
// It is not bound behind the L2s: at 301 rows gate/up fetches 200 MB, 1.10 times its operands.
// Cold weights, against the kernels that took these sizes before (folds included), microseconds at 161 / 301 / 552 rows: 7B
// gate/up 91 -> 47 / 94 -> 65 / 121 -> 110, the other three 109 -> 68 / 153 -> 106 / 220 -> 144; 8B-GQA gate/up 99 -> 54 /
// 103 -> 77 / 162 -> 127, the other three 101 -> 65 / 136 -> 95 / 184 -> 142.
//
// A ring of as many whole stages (activations + weights of one 64-wide k-tile) as the CU's LDS holds, filled by
// direct global->LDS loads.  The barrier of tile i sits between its two k-steps, whose second one runs from
// registers: from there on tile i's stage is free, and tile i + kStages is requested into it over the following
// two k-steps, so kStages - 2 whole tiles stay in flight across every barrier.  Operands of the next k-step are
// read from LDS under the MFMAs of the present one.
// ---------------------------------------------------------------------------------------------
template <int WT, int NBT, int NBF> struct MidCfg {
    static constexpr int WF = 4 / WT;
    static constexpr int BM = WT * NBT * 16, BN = WF * NBF * 16;
    static constexpr int kXBytes = BM * kBK * (int)sizeof(bf16);
    static constexpr int kStage = (BM + BN) * kBK * (int)sizeof(bf16);
    static constexpr int kFit = 160 * 1024 / kStage;
    static constexpr int kStages = kFit < 5 ? kFit : 5;
    static constexpr int kLds = kStage * kStages;
    static_assert(NBF % 2 == 0 && BM % 32 == 0 && kStages >= 2, "tile");
};

// vmcnt(n) lgkmcnt(0), n < 64
__device__ __forceinline__ constexpr int lds_wait(int n) { return ((n >> 4) << 14) | 0x0070 | (n & 15); }

// GU (gate/up projection): weight rows come as N gate rows, then N up rows; a tile takes BN / 2 features, and of every
// 32 LDS rows 16 hold gate and 16 the same features' up rows, so a lane holds both factors.
// `partial` != nullptr: fp32 partial sums partial[range][M][Nrows]; else C, with the residual R unless null.
template <bool GU, bool NT, int WT, int NBT, int NBF>
__global__ __launch_bounds__(256, 1) void gemm_mid_kernel(const bf16* __restrict__ X, const bf16* __restrict__ W,
                                                          float* __restrict__ partial, const bf16* R, bf16* C, int M,
                                                          int Nrows, int K, int n_tiles, int m_tiles, int kt_per_split,
                                                          int units) {
    using Cfg = MidCfg<WT, NBT, NBF>;
    constexpr int BM = Cfg::BM, BN = Cfg::BN, S = Cfg::kStages;
    constexpr int PX = BM / 32, PW = BN / 32, P = PX + PW;      // 1 KiB pieces (8 rows) a wave requests per k-tile
    constexpr int NMMA = NBT * NBF, NFETCH = NBT + NBF;
    static_assert((S - 1) * P < 64, "loads in flight must be countable");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    // A unit is one (weight tile, K range); its m_tiles workgroups get ids 8 apart, hence one XCD, one after the
    // other, so that the later ones find the weights in that XCD's L2.
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    const int unit = (seq / m_tiles) * 8 + xcd;
    if (unit >= units) return;
    const int m0 = (seq % m_tiles) * BM;
    const int tile_n = unit % n_tiles, split = unit / n_tiles;
    const int Nh = Nrows >> 1;                                  // GU: features per factor
    const int n0 = tile_n * (GU ? BN / 2 : BN);
    const int nk = K / kBK;
    const int kt0 = split * kt_per_split;
    const int kt1 = (kt0 + kt_per_split < nk) ? kt0 + kt_per_split : nk;
    const int n = kt1 - kt0;                                    // >= 1

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wt = wave % WT, wf = wave / WT;
    const int lrow = lane & 15, lg = lane >> 4;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);

    uint32_t x_off[PX], w_off[PW];
#pragma unroll
    for (int j = 0; j < PX; ++j) {
        const int row = (wave * PX + j) * 8 + (lane >> 3);
        int xr = m0 + row;
        if (xr > M - 1) xr = M - 1;
        x_off[j] = ((uint32_t)xr * (uint32_t)K + ((lane & 7) ^ swz(row)) * 8) * 2u;
    }
#pragma unroll
    for (int j = 0; j < PW; ++j) {
        const int row = (wave * PW + j) * 8 + (lane >> 3);
        int wr;
        if (GU) {
            int f = n0 + (row >> 5) * 16 + (row & 15);
            if (f > Nh - 1) f = Nh - 1;
            wr = (row & 16) ? Nh + f : f;
        } else {
            wr = n0 + ((row & ~31) | big_row_feature(row & 31));
            if (wr > Nrows - 1) wr = Nrows - 1;
        }
        w_off[j] = ((uint32_t)wr * (uint32_t)K + ((lane & 7) ^ swz(row)) * 8) * 2u;
    }
    const __amdgpu_buffer_rsrc_t rsrc_x =
        __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, (int)((uint32_t)M * (uint32_t)K * 2u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w =
        __builtin_amdgcn_make_buffer_rsrc((void*)W, 0, (int)((uint32_t)Nrows * (uint32_t)K * 2u), 0x00020000);
    // piece q of the k-tile at byte offset `koff` into stage `st`: weights (from memory) first, then activations
    auto issue_piece = [&](int koff, unsigned char* st, int q) {
        if (q < PW)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w, (lptr_t)(st + Cfg::kXBytes + (wave_u * PW + q) * 1024), 16,
                                                     (int)w_off[q], koff, 0, NT ? 2 : 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (lptr_t)(st + (wave_u * PX + q - PW) * 1024), 16,
                                                     (int)x_off[q - PW], koff, 0, 0);
    };

    f32x4 acc[NBF][NBT];
#pragma unroll
    for (int j = 0; j < NBF; ++j)
#pragma unroll
        for (int i = 0; i < NBT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][i][r] = 0.f;

    int xk[2], wk[2];                                           // operand addresses inside a stage, per k-step
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int piece = ((ks * 4 + lg) ^ swz(lrow)) * 16;
        xk[ks] = (wt * NBT * 16 + lrow) * 128 + piece;
        wk[ks] = Cfg::kXBytes + (wf * NBF * 16 + lrow) * 128 + piece;
    }
    bf16x8 xf[2][NBT], wfr[2][NBF];
    auto fetch = [&](const unsigned char* st, int ks, int buf, int q) {        // in the order of first use
        if (q == 0) wfr[buf][0] = *reinterpret_cast<const bf16x8*>(st + wk[ks]);
        else if (q <= NBT) xf[buf][q - 1] = *reinterpret_cast<const bf16x8*>(st + xk[ks] + (q - 1) * 2048);
        else wfr[buf][q - NBT] = *reinterpret_cast<const bf16x8*>(st + wk[ks] + (q - NBT) * 2048);
    };
    // One k-step: the MFMAs from buffer `cur`; between them the LDS reads of k-step `nks` of stage `st` into the other
    // buffer, over the first three quarters, and the requests for pieces q0 .. q1 - 1, spread evenly.
    auto kstep = [&](auto cur_, auto fetch_, const unsigned char* st, int nks, auto issue_, int koff, unsigned char* dst,
                     int q0, int q1) {
        constexpr int cur = decltype(cur_)::value;
        constexpr bool do_fetch = decltype(fetch_)::value, do_issue = decltype(issue_)::value;
        __builtin_amdgcn_sched_barrier(0);
        auto fetch_upto = [](int q) { return q < 0 ? 0 : ((q + 1) * NFETCH * 4 + 3 * NMMA - 1) / (3 * NMMA); };
        auto issue_upto = [&](int q) { return q0 + ((q + 1) * (q1 - q0)) / NMMA; };
#pragma unroll
        for (int q = 0; q < NMMA; ++q) {
            acc[q / NBT][q % NBT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfr[cur][q / NBT], xf[cur][q % NBT],
                                                                          acc[q / NBT][q % NBT], 0, 0, 0);
            if (do_fetch) {
#pragma unroll
                for (int f = 0; f < NFETCH; ++f)
                    if (f >= fetch_upto(q - 1) && f < fetch_upto(q)) fetch(st, nks, cur ^ 1, f);
            }
            if (do_issue) {
#pragma unroll
                for (int f = 0; f < P; ++f)
                    if (f >= issue_upto(q - 1) && f < issue_upto(q)) issue_piece(koff, dst, f);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // all but the newest `tiles` k-tiles requested have landed, own LDS reads are done; then everyone's
    auto wait_barrier = [&](int tiles) {
        if (S > 4 && tiles >= 4) __builtin_amdgcn_s_waitcnt(lds_wait(S > 4 ? 4 * P : 0));
        else if (S > 3 && tiles == 3) __builtin_amdgcn_s_waitcnt(lds_wait(S > 3 ? 3 * P : 0));
        else if (S > 2 && tiles == 2) __builtin_amdgcn_s_waitcnt(lds_wait(S > 2 ? 2 * P : 0));
        else if (tiles == 1) __builtin_amdgcn_s_waitcnt(lds_wait(P));
        else __builtin_amdgcn_s_waitcnt(lds_wait(0));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using Yes = std::true_type;
    using No = std::false_type;

    // The walk over K does not start at the first k-tile everywhere, or the whole chip would read one column of all weight rows
    // at a time, which crowds onto few memory channels.  With one row of tiles it starts tile_n / n_tiles of the way in when the
    // row pitch is a power of two, as in the decode kernel below (161 rows: 7B gate/up 47.4 -> 44.7 us, 8B-GQA 55.7 -> 51.7).
    // With several, the workgroups that share a weight tile and those that share activations do better in step (552 rows: 8B-GQA
    // qkv 34.5 in step, 40.8 shifted each by itself), so with two or three each XCD, where the sharing is, has one start (three layers of
    // the 7B shape, 301 rows 605 -> 586 us, 250 rows 549 -> 542, two of 70B, 250 rows 1008 -> 1002; two starts per XCD the same); with
    // more, all are in step (shifted by XCD, 13B 700 rows 991 -> 995, 8B-GQA 1200 rows 1548 -> 1553).
    // They also are where the pitch is a power of two and neighbouring tiles lie 2^11 or 2^8 times as far apart as the starts (of a KiB
    // and more), or 2 MiB (starts of more than 512 bytes): the two differences then cancel in the choice of the channel.  Shifted against in step, cold weights:
    // 8192 rows of 8192 at 257 rows 55.8 -> 61.8 us, 28672 of 4096 at 270 rows 76.1 -> 85.5, gate/up of 4096 features of 8192 at 240 rows
    // 55.3 -> 63.2, of 8192 of 16384 at 330 rows 186 -> 199 (2 MiB; 70B gate/up 0 to 1.7 % there).  Other orders of the eight starts
    // lose elsewhere.  And they are from eight ranges of K on, whose workgroups are at eight places anyway (2048 rows of 16384 at 390 rows
    // 45.4 -> 49.2).  Over the 1300 other products of 2 or 3 rows of tiles that were measured shifted takes 0.96 to 0.985 of the time.
    constexpr int kApart = GU ? BN / 2 : BN;                    // weight rows between neighbouring tiles
    const long long apart = (long long)kApart * K;              // starts: n / 8 k-tiles of 64 columns
    const bool cancel = (K & (K - 1)) == 0 &&
                        ((n >= 64 && (apart == (long long)n << 14 || apart == (long long)n << 11)) || (n > 32 && apart == 1 << 20));
    const int rot = n < 32 || m_tiles > 3 || (m_tiles > 1 && (cancel || n * 8 <= nk)) ? 0 : m_tiles > 1 ? xcd * n / 8 : (K & (K - 1)) == 0 ? (int)(((long long)tile_n * n) / n_tiles) : 0;
    auto koff_of = [&](int j) { const int r = j + rot; return (kt0 + (r >= n ? r - n : r)) * (kBK * 2); };
    const int first = n < S ? n : S;
#pragma unroll
    for (int t = 0; t < S; ++t)
        if (t < n) {
            const int koff = koff_of(t);
#pragma unroll
            for (int q = 0; q < P; ++q) issue_piece(koff, smem_raw + t * Cfg::kStage, q);
        }
    wait_barrier(first - 1);
#pragma unroll
    for (int q = 0; q < NFETCH; ++q) fetch(smem_raw, 0, 0, q);
    kstep(C0(), Yes(), smem_raw, 1, No(), 0, smem_raw, 0, 0);
    int s = 0;
    int i = 0;
    for (; i < n - S; ++i) {
        wait_barrier(S - 2);
        const int nx = s + 1 == S ? 0 : s + 1;
        const int koff = koff_of(i + S);
        const unsigned char* next = smem_raw + nx * Cfg::kStage;
        unsigned char* dst = smem_raw + s * Cfg::kStage;
        kstep(C1(), Yes(), next, 0, Yes(), koff, dst, 0, (P + 1) / 2);
        kstep(C0(), Yes(), next, 1, Yes(), koff, dst, (P + 1) / 2, P);
        s = nx;
    }
    for (; i < n - 1; ++i) {
        wait_barrier(n - 2 - i);
        const int nx = s + 1 == S ? 0 : s + 1;
        const unsigned char* next = smem_raw + nx * Cfg::kStage;
        kstep(C1(), Yes(), next, 0, No(), 0, smem_raw, 0, 0);
        kstep(C0(), Yes(), next, 1, No(), 0, smem_raw, 0, 0);
        s = nx;
    }
    kstep(C1(), No(), smem_raw, 0, No(), 0, smem_raw, 0, 0);
    __builtin_amdgcn_sched_barrier(0);

    // A lane holds, of token block i, token i*16 + lane%16, and of block pair p either 8 consecutive weight rows or
    // (GU) 4 consecutive features of both factors.
#pragma unroll
    for (int i = 0; i < NBT; ++i) {
        const int m = m0 + (wt * NBT + i) * 16 + lrow;
        if (m < M) {
            if (partial != nullptr) {
                float* prow = partial + ((size_t)split * M + m) * Nrows;
#pragma unroll
                for (int p = 0; p < NBF / 2; ++p) {
                    if (GU) {
                        const int f = n0 + (wf * (NBF / 2) + p) * 16 + 4 * lg;
                        if (f < Nh) {
                            *reinterpret_cast<f32x4*>(prow + f) = acc[2 * p][i];
                            *reinterpret_cast<f32x4*>(prow + Nh + f) = acc[2 * p + 1][i];
                        }
                    } else {
                        const int f = n0 + wf * NBF * 16 + p * 32 + 8 * lg;
                        if (f < Nrows) *reinterpret_cast<f32x4*>(prow + f) = acc[2 * p][i];
                        if (f + 4 < Nrows) *reinterpret_cast<f32x4*>(prow + f + 4) = acc[2 * p + 1][i];
                    }
                }
            } else if (GU) {
                bf16* crow = C + (size_t)m * Nh;
#pragma unroll
                for (int p = 0; p < NBF / 2; ++p) {
                    const int f = n0 + (wf * (NBF / 2) + p) * 16 + 4 * lg;
                    bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (bf16)(silu_fast(acc[2 * p][i][e]) * acc[2 * p + 1][i][e]);
                    if (f < Nh) *reinterpret_cast<bf16x4*>(crow + f) = o;
                }
            } else {
                // R may be C itself: a token's residual values are read before its results are written
                bf16x8 rv[NBF / 2];
                if (R != nullptr) {
#pragma unroll
                    for (int p = 0; p < NBF / 2; ++p)
                        rv[p] = big_load8(R + (size_t)m * Nrows, n0 + wf * NBF * 16 + p * 32 + 8 * lg, Nrows);
                }
#pragma unroll
                for (int p = 0; p < NBF / 2; ++p) {
                    float o[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        o[e] = acc[2 * p + (e >> 2)][i][e & 3];
                        if (R != nullptr) o[e] += (float)rv[p][e];
                    }
                    big_store8(C + (size_t)m * Nrows, n0 + wf * NBF * 16 + p * 32 + 8 * lg, Nrows, o);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Tiles that exist.  Chosen so that over 65 .. 1600 rows of six projection shapes the best of them is within 1 % of the
// best of 34 measured; 320 x 96 is the fastest on none of 596 problems and no longer among them.
struct MidTile { int wt, nbt, nbf; };
#define BZ_MID_TILES(X) X(2, 3, 4) X(4, 2, 4) X(4, 2, 6) X(4, 3, 6) X(4, 3, 8) X(2, 5, 4) X(2, 5, 6) X(2, 6, 6) X(2, 7, 6) \
                        X(2, 5, 8) X(2, 8, 4) X(4, 4, 6)
constexpr MidTile kMidTiles[] = {
#define BZ_MID_ENTRY(a, b, c) {a, b, c},
    BZ_MID_TILES(BZ_MID_ENTRY)
#undef BZ_MID_ENTRY
};
constexpr int kMidMinM = 65, kMidMaxM = 2048;
constexpr size_t kMidMaxPartial = BZ_STATIC_SCRATCH_BYTES;      // partial sums stay within the static scratch

struct MidPlan {
    int tile, m_tiles, n_tiles, kt_per_split, ksplit;
    float us;                    // what the model expects, with the cost of folding the partial sums
    size_t ws_bytes;
};

// Time model, microseconds, fitted to 26 000 measurements with cold weights (596 problems of 65 to 1938 rows, all tiles, 1 to 16
// ranges; 9 % rms).  A k-tile costs 0.043 + 0.00069 BM + 0.00124 BN + 8.8e-6 BM BN; a round 1.35, and 0.066 per MB of activations
// that the eight XCDs fetch in it; the weights stream at 7.15 TB/s at most, and the two bound the body together (4-norm).
// Partial sums cost 0.434 per MB and, behind gate/up, 1.8 for the kernel that folds them (elsewhere the next step does).
// A round is what an XCD's 32 CUs hold: an XCD takes whole units, so 27 units of 9 tiles (243 workgroups) are two rounds,
// four units being 36 workgroups on three of the XCDs.  Against the kernels of before (65 to 256 rows the decode kernel in
// blocks of 128, beyond the large tiles) the plans are 20 % faster on average and slower by more than 4 % on 16 of the 596.
// An earlier model, without rounds per XCD and the cost of many rows sharing few weights, picked plans slower than those
// kernels on 67 of them (70B down projection at 65 to 128 rows 139 -> 84 us with this one, 13B at 398 rows 109 -> 73).
// `room`: bytes of scratch there are; the best plan within them.
static MidPlan mid_plan(int mode, int M, int N, int K, size_t room) {
    const int Nrows = (mode == 2) ? 2 * N : N, nk = K / kBK;
    constexpr int kCUs = 256, kMinKt = 4;
    MidPlan best{};
    best.us = -1.f;
    for (int t = 0; t < (int)(sizeof(kMidTiles) / sizeof(kMidTiles[0])); ++t) {
        const int bm = kMidTiles[t].wt * kMidTiles[t].nbt * 16, bn = (4 / kMidTiles[t].wt) * kMidTiles[t].nbf * 16;
        const int mt = (M + bm - 1) / bm, nt = (Nrows + bn - 1) / bn;
        const float tk = 0.043f + 0.69e-3f * (float)bm + 1.24e-3f * (float)bn + 8.8e-6f * (float)(bm * bn);
        int most = kCUs / (mt * nt);
        if (most > 16) most = 16;
        if (most > nk / kMinKt) most = nk / kMinKt;
        for (int ks = 1; ks == 1 || ks <= most; ++ks) {
            const int per = (nk + ks - 1) / ks;
            if ((nk + per - 1) / per != ks) continue;           // same ranges as a smaller number of them
            const size_t bytes = ks > 1 ? (size_t)ks * M * Nrows * sizeof(float) : 0;
            if (bytes > kMidMaxPartial || bytes > room) break;
            const int rounds = ((nt * ks + 7) / 8 * mt + kCUs / 8 - 1) / (kCUs / 8);
            const float fetched = (float)rounds * 8.f * (float)M * (float)K * 2.f / (float)ks;
            const float body = (float)rounds * (float)per * tk + 0.066e-6f * fetched;
            const float stream = (float)Nrows * (float)K * 2.f / 7.15e6f;
            const float b2 = body * body, s2 = stream * stream;
            const float us = 8.0f + sqrtf(sqrtf(b2 * b2 + s2 * s2)) + 1.35f * (float)rounds + 0.434e-6f * (float)bytes +
                             (ks > 1 ? (mode == 2 ? 1.8f : 0.5f) : 0.f);
            if (best.us < 0.f || us < best.us) best = MidPlan{t, mt, nt, per, ks, us, bytes};
        }
    }
    return best;
}

// The large-tile kernel on the same scale: a k-tile costs 0.88, and up to 0.51 more the more of the CUs a round fills; split
// tiles add a fix-up launch and their traffic.
static float big_us(int mode, int M, int N, int K) {
    const BigPlan p = big_plan(mode, M, N, K);
    const float nk = (float)(K / kBK);
    float body = 0.f;
    if (p.n_dp > 0) {
        const float rounds = (float)((p.n_dp + 255) / 256);
        body = rounds * (nk * (0.88f + 0.51f * (float)p.n_dp / (256.f * rounds)) + 11.4f);
    }
    if (p.tail > 0)
        body += (float)((K / kBK + p.splits - 1) / p.splits) * (0.88f + 0.51f * (float)(p.tail * p.splits) / 256.f) + 12.5f +
                (float)p.ws_bytes * 0.162e-6f;
    const float us = 1.5f + body, stream = 1.5f + (float)((mode == 2) ? 2 * N : N) * (float)K * 2.f / 5.07e6f;
    const float b2 = us * us, s2 = stream * stream;
    return sqrtf(sqrtf(b2 * b2 + s2 * s2));
}

// Whether the mid-sized kernel takes the problem: always up to 256 rows (the large tiles win on one of 274 problems there, by
// 5 %), beyond unless the models see the large tiles 5 % ahead.  Over the 596 problems the choice costs
// 1.8 % against the best of all forms (without the margin as much on average, with more calls slower than before).
// Which kernel is a matter of the shape alone; `p` is the plan within the scratch there is.
static bool mid_takes(int mode, int M, int N, int K, size_t room, MidPlan& p) {
    if (M < kMidMinM || M > kMidMaxM || !big_ok(M, N, K)) return false;
    p = mid_plan(mode, M, N, K, kMidMaxPartial);
    if (M > 256 && p.us >= 0.95f * big_us(mode, M, N, K)) return false;
    if (p.ws_bytes > room) p = mid_plan(mode, M, N, K, room);
    return true;
}

struct MidArgs {
    const bf16* x; const bf16* w; float* partial; const bf16* r; bf16* c;
    int M, Nrows, K, n_tiles, m_tiles, kt_per_split, units;
};

// false: the runtime does not grant the kernel its LDS
template <bool GU, int WT, int NBT, int NBF>
static bool mid_go(hipStream_t st, const MidArgs& g) {
    using Cfg = MidCfg<WT, NBT, NBF>;
    const dim3 grid((g.units + 7) / 8 * 8 * g.m_tiles);
    // weights that one workgroup reads and nobody else are loaded with the non-temporal policy (1.5 - 3 % at 65 .. 301 rows)
    if (g.m_tiles == 1) {
        static LdsLimit limit;
        if (!limit.raise(reinterpret_cast<const void*>(gemm_mid_kernel<GU, true, WT, NBT, NBF>), Cfg::kLds)) return false;
        hipLaunchKernelGGL((gemm_mid_kernel<GU, true, WT, NBT, NBF>), grid, dim3(256), Cfg::kLds, st, g.x, g.w, g.partial, g.r,
                           g.c, g.M, g.Nrows, g.K, g.n_tiles, g.m_tiles, g.kt_per_split, g.units);
    } else {
        static LdsLimit limit;
        if (!limit.raise(reinterpret_cast<const void*>(gemm_mid_kernel<GU, false, WT, NBT, NBF>), Cfg::kLds)) return false;
        hipLaunchKernelGGL((gemm_mid_kernel<GU, false, WT, NBT, NBF>), grid, dim3(256), Cfg::kLds, st, g.x, g.w, g.partial, g.r,
                           g.c, g.M, g.Nrows, g.K, g.n_tiles, g.m_tiles, g.kt_per_split, g.units);
    }
    return true;
}

// Partial sums into `ws` when the plan has several ranges of K, else the result itself into `c` (r: the residual or null).
static bool launch_mid(int mode, const MidPlan& p, const bf16* x, const bf16* w, const bf16* r, bf16* c, int M, int N, int K,
                       float* ws, hipStream_t st) {
    using Fn = bool (*)(hipStream_t, const MidArgs&);
#define BZ_MID_FN(a, b, c) mid_go<false, a, b, c>,
#define BZ_MID_FN_GU(a, b, c) mid_go<true, a, b, c>,
    static constexpr Fn plain[] = {BZ_MID_TILES(BZ_MID_FN)};
    static constexpr Fn gated[] = {BZ_MID_TILES(BZ_MID_FN_GU)};
#undef BZ_MID_FN
#undef BZ_MID_FN_GU
    const MidArgs g{x, w, p.ksplit > 1 ? ws : nullptr, mode == 1 ? r : nullptr, c, M, (mode == 2) ? 2 * N : N, K,
                    p.n_tiles, p.m_tiles, p.kt_per_split, p.n_tiles * p.ksplit};
    return (mode == 2 ? gated : plain)[p.tile](st, g);
}

// ---------------------------------------------------------------------------------------------
// Skinny kernel for decode-sized problems (M <= 64 rows): the weights are read from HBM exactly
// once and that read is the whole cost, so the job is to keep every CU streaming.  Work is cut
// into tiles of 64 * RB weight rows times KSPLIT slices of K (a function of the shape only); each
// workgroup streams its weight slice and the matching activation slice through a ring of LDS
// stages filled by direct global->LDS loads, multiplies with RB 32x32x16 MFMAs per wave and
// k-step, and writes an fp32 partial tile.  A second kernel adds the slices in slice order and
// applies the epilogue, so the result is deterministic.
//
// RB = 1: 64-row tiles, four 16 KiB stages, two workgroups per CU: short streams (small matrices),
// where many small workgroups start and finish faster.
// RB = 2: 128-row tiles: long streams.  Every tile re-reads the activations from L2, which costs about a tenth of the time at 64
// rows; twice the rows halve that.  Workgroups per CU: two with TB = 1 (four 20 KiB stages), one with TB = 2 and four 24 KiB stages,
// two with three of them.  Measured against RB = 1 on the decode shapes (64 rows, five stages): 8B-GQA down projection 31.4 -> 28.0 us, gate/up
// unchanged; 70B qkv 40.9 -> 37.1, o 36.1 -> 37.8, gate/up 185 -> 168, down 96.5 -> 78.5 us.
//
// TB: 32-row blocks of the activations in a stage; with one (up to 32 rows) the four waves share out the weight rows alone.
// ST: stages.  A stage of 64 activation rows costs as many loads whether they are real or not, and behind 32 real ones
// half of them; four stages are better than five or seven, in either form.  Us at 32 rows: 70B gate/up 161 -> 148, down 77.2 ->
// 75.3, qkv 32.0 -> 30.2, o 26.8 -> 25.5; at 20 rows: 13B 47.7 -> 45.4, 28.8 -> 27.5 (qkv), 25.9 -> 24.6 (down); at 12: 7B 34.4 ->
// 29.6 (with the tiles as many as CUs, below), 19.2 -> 17.7, 18.7 -> 17.6; at 24: 8B-GQA 37.1 -> 36.4, 20.6 -> 20.4.  Above 32 rows four
// stages instead of five: 13B (48) 49.9 -> 49.5, 30.9 -> 30.4, 27.2 -> 26.7, 7B gate/up (64) 36.8 -> 35.5.  Where there are more
// tiles than CUs three, which leave room for two workgroups: 70B gate/up (64) 172 -> 161; elsewhere they lose (13B 52.5, 31.1, 27.6).
template <int RB, int TB, int ST> struct SkCfg {
    static constexpr int kXBytes = 32 * TB * kBK * (int)sizeof(bf16);         // activations of a stage: 4 KiB * TB
    static constexpr int kStage = kXBytes + 64 * RB * kBK * (int)sizeof(bf16);  // + weights 8 KiB * RB
    static constexpr int kStages = ST;
    static constexpr int kLds = kStage * kStages;
    static constexpr int kPerCu = kLds * 2 <= 160 * 1024 ? 2 : 1;
};
// Weight matrices from this size on count as long streams: RB = 2, and loads with the non-temporal cache
// policy (read once per step; streamed that way a long read runs faster - gate/up of the 8B shape -6 % -
// a short one does not or gets slower).
constexpr size_t kSkStreamBytes = (size_t)64 << 20;

// GU (gate/up projection): a tile is 32 * RB gate features (weight rows n0..) and the matching up
// features (rows N + n0..), so that with a single k-slice the workgroup holds both factors of
// silu(gate) * up and writes the activation itself (C != nullptr) instead of partial sums.
// NT: the weight loads carry the non-temporal cache policy.
// TAIL: K is a multiple of 8 and not of 64.  The last k-tile's pieces past the end re-read the row's last piece and count as
// zero, both operands, when they are multiplied.  (Such shapes went to the 64x128 kernel before, with a workgroup per 128
// weight rows and K uncut: 688 -> 256 at one row 10.0 -> 4.8 us.)
template <bool GU, bool NT, int RB, int TB, int ST, bool TAIL>
__global__ __launch_bounds__(256, (SkCfg<RB, TB, ST>::kPerCu)) void gemm_skinny_kernel(const bf16* __restrict__ X,
                                                                             const bf16* __restrict__ W,
                                                                             float* __restrict__ partial,
                                                                             bf16* __restrict__ C, int M, int Nrows, int K,
                                                                             int n_tiles, int kt_per_split, int rows) {
    using Cfg = SkCfg<RB, TB, ST>;
    constexpr int kStage = Cfg::kStage, kStages = Cfg::kStages, kXBytes = Cfg::kXBytes;
    constexpr int LPS = TB + 2 * RB;                  // loads per wave and stage
    constexpr int NB = TB == 2 ? RB : RB / 2;         // 32-row blocks of a wave
    static_assert(NB >= 1, "TB = 1: the four waves share out the weight rows alone");
    static_assert(kStages == 3 || kStages == 4, "the waits count up to two later tiles");
    constexpr int HALF = 32 * RB;                     // rows per wave along the features (GU: rows per factor)
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const int tile_n = blockIdx.x % n_tiles, split = blockIdx.x / n_tiles;
    // `rows` <= 64 * RB weight rows of those the tile has room for are real (GU: rows / 2 of each factor);
    // the launcher picks it so that the grid fills the chip's workgroup slots evenly
    const int tr = GU ? rows >> 1 : rows;             // real rows per factor (GU) or per tile
    const int n0 = tile_n * tr;
    const int Nh = Nrows >> 1;                        // GU: features per factor
    const int nk = (K + kBK - 1) / kBK;
    const int kt0 = split * kt_per_split;
    const int kt1 = (kt0 + kt_per_split < nk) ? kt0 + kt_per_split : nk;
    const int n = kt1 - kt0;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wf = wave >> 1, wt = TB == 2 ? wave & 1 : 0;          // feature half, token half
    const int b0 = TB == 2 ? 0 : (wave & 1) * NB;                   // first block of the half's RB
    const int lrow = lane & 31, lk = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);

    // loader: 1 KiB chunks of 8 rows; the first 4 * TB chunks of a stage hold the activation rows, the
    // 8 * RB after them the weight rows; this wave fills TB of the former and 2 * RB of the latter
    uint32_t x_src[TB], w_src[2 * RB];
#pragma unroll
    for (int j = 0; j < TB; ++j) {
        const int row = (wave * TB + j) * 8 + (lane >> 3);
        int xr = row;
        if (xr > M - 1) xr = M - 1;
        x_src[j] = ((uint32_t)xr * (uint32_t)K + ((lane & 7) ^ swz(row)) * 8) * 2u;
    }
#pragma unroll
    for (int j = 0; j < 2 * RB; ++j) {
        const int row = (wave * 2 * RB + j) * 8 + (lane >> 3);
        int wr;
        if (GU) {                                      // rows past the real ones re-read the tile's last row
            int r = row % HALF;
            if (r > tr - 1) r = tr - 1;
            int f = n0 + r;
            if (f > Nh - 1) f = Nh - 1;
            wr = (row / HALF) * Nh + f;
        } else {
            wr = n0 + (row < tr ? row : tr - 1);
            if (wr > Nrows - 1) wr = Nrows - 1;
        }
        w_src[j] = ((uint32_t)wr * (uint32_t)K + ((lane & 7) ^ swz(row)) * 8) * 2u;
    }
    auto issue = [&](int kt, int stage) {
        const char* xk = reinterpret_cast<const char*>(X + (size_t)kt * kBK);
        const char* wk = reinterpret_cast<const char*>(W + (size_t)kt * kBK);
        unsigned char* sb = smem_raw + stage * kStage;
        const int left = TAIL ? K - kt * kBK : kBK;      // columns the tile has; a multiple of 8
        // bytes by which a lane's piece of LDS row `row` lies behind the row's last one
        auto back = [&](int row) {
            const int c = ((lane & 7) ^ swz(row)) * 8;
            return TAIL && c >= left ? (uint32_t)(c - (left - 8)) * 2u : 0u;
        };
#pragma unroll
        for (int j = 0; j < TB; ++j)
            __builtin_amdgcn_global_load_lds((gptr_t)(xk + x_src[j] - back((wave * TB + j) * 8 + (lane >> 3))),
                                             (lptr_t)(sb + (wave_u * TB + j) * 1024), 16, 0, 0);
#pragma unroll
        for (int j = 0; j < 2 * RB; ++j)
            __builtin_amdgcn_global_load_lds((gptr_t)(wk + w_src[j] - back((wave * 2 * RB + j) * 8 + (lane >> 3))),
                                             (lptr_t)(sb + kXBytes + (wave_u * 2 * RB + j) * 1024), 16, 0, NT ? 2 : 0);
    };

    f32x16 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
    const int sw = swz(lrow);
    const int x_off = (wt * 32 + lrow) * 128;
    const int w_off = kXBytes + (wf * HALF + b0 * 32 + lrow) * 128;

    // Every workgroup would walk its k-tiles in the same order at about the same pace, so that at any moment the
    // whole chip reads the same 128-byte column of thousands of weight rows; when the row pitch is a power of two
    // those addresses differ in their high bits only and crowd onto few memory channels.  A tile therefore starts
    // its walk tile_n / n_tiles of the way in and wraps around (a function of the shape and the tile alone, so
    // the sum order, and with it every output bit, stays fixed).  Measured in the decode loop: gate/up of the 8B
    // shape 50 -> 41 us, output projection of the 70B shape 32 -> 26 us, its QKV 34 -> 32 us; pitches that are
    // no power of two, and walks of fewer than 32 tiles, gain nothing or lose 1-2 % and keep the plain order.
    const int rot = ((K & (K - 1)) == 0 && n >= 32) ? (int)(((long long)tile_n * n) / n_tiles) : 0;
    auto kmap = [&](int j) { const int r = j + rot; return kt0 + (r >= n ? r - n : r); };   // j-th k-tile of the walk
    // prologue: up to kStages - 1 tiles in flight
#pragma unroll
    for (int t = 0; t < kStages - 1; ++t)
        if (n > t) issue(kmap(t), t);
    int cur = 0, nxt = kStages - 1;                  // stage of tile i; stage the tile requested next goes to
    for (int i = 0; i < n; ++i) {
        // tile i must have landed; the tiles requested after it (LPS loads each) may still be in flight
        const int later = (n - 1 - i < kStages - 2) ? n - 1 - i : kStages - 2;
        if (later == 2) __builtin_amdgcn_s_waitcnt(lds_wait(2 * LPS));
        else if (later == 1) __builtin_amdgcn_s_waitcnt(lds_wait(LPS));
        else __builtin_amdgcn_s_waitcnt(lds_wait(0));
        __builtin_amdgcn_s_barrier();                              // everyone's part landed; the stage of tile i-1 is free
        __builtin_amdgcn_sched_barrier(0);
        if (i + kStages - 1 < n) issue(kmap(i + kStages - 1), nxt);
        const unsigned char* st = smem_raw + cur * kStage;
        nxt = cur;
        cur = (cur + 1 == kStages) ? 0 : cur + 1;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int ko = ((ks * 2 + lk) ^ sw) * 16;
            bf16x8 xf = *reinterpret_cast<const bf16x8*>(st + x_off + ko);
            const bool past = TAIL && kmap(i) * kBK + (ks * 2 + lk) * 8 >= K;
            if (past) xf = bf16x8{};
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                bf16x8 wfr = *reinterpret_cast<const bf16x8*>(st + w_off + b * 32 * 128 + ko);
                if (past) wfr = bf16x8{};
                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfr, xf, acc[b], 0, 0, 0);
            }
        }
    }

    // lane holds token wt*32 + lane%32 and, of block b of its wave's rows, features 8g + 4*(lane/32) + 0..3
    const int m = wt * 32 + lrow;
    if (GU && C != nullptr) {
        // the up-factor waves hand their accumulators to the gate-factor waves (same lane, same
        // token half) through LDS, which is free once everyone has read the last stage
        float* ex = reinterpret_cast<float*>(smem_raw);
        __syncthreads();
        if (wf == 1) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) ex[((wt * RB + b0 + b) * 16 + r) * 64 + lane] = acc[b][r];
        }
        __syncthreads();
        if (wf == 0 && m < M) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int lf = (b0 + b) * 32 + 8 * g + 4 * lk;
                    const int nn = n0 + lf;
                    if (lf < tr && nn < Nh) {
                        bf16x4 w4;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float o = acc[b][4 * g + e];
                            const float u = ex[((wt * RB + b0 + b) * 16 + 4 * g + e) * 64 + lane];
                            w4[e] = (bf16)(silu_fast(o) * u);
                        }
                        *reinterpret_cast<bf16x4*>(C + (size_t)m * Nh + nn) = w4;
                    }
                }
        }
        return;
    }
    if (m >= M) return;
    float* prow = partial + ((size_t)split * M + m) * Nrows;           // partial[split][m][n]
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int lf = (GU ? 0 : wf * HALF) + (b0 + b) * 32 + 8 * g + 4 * lk;      // feature inside the tile (GU: the factor)
            const int f = n0 + lf;
            const int nn = GU ? wf * Nh + f : f;
            if (lf < tr && f < (GU ? Nh : Nrows))
                *reinterpret_cast<float4*>(prow + nn) =
                    make_float4(acc[b][4 * g], acc[b][4 * g + 1], acc[b][4 * g + 2], acc[b][4 * g + 3]);
        }
}

template <int MODE>
__global__ __launch_bounds__(256) void gemm_partial_epilogue(const float* __restrict__ partial, const bf16* R, bf16* C,
                                                            int M, int N, int Nrows, int ksplit) {
    const int idx = blockIdx.x * 256 + threadIdx.x;       // one thread per 4 outputs
    const int per_row = N >> 2;
    if (idx >= M * per_row) return;
    const int m = idx / per_row, n = (idx - m * per_row) * 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f), u = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < ksplit; ++k) {
        const float* prow = partial + ((size_t)k * M + m) * Nrows;
        const float4 a = *reinterpret_cast<const float4*>(prow + n);
        s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
        if (MODE == 2) {
            const float4 b = *reinterpret_cast<const float4*>(prow + N + n);
            u.x += b.x; u.y += b.y; u.z += b.z; u.w += b.w;
        }
    }
    float o[4] = {s.x, s.y, s.z, s.w};
    if (MODE == 1) {
        const bf16x4 rv = *reinterpret_cast<const bf16x4*>(R + (size_t)m * N + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] += (float)rv[e];
    }
    if (MODE == 2) {
        const float uu[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = silu_fast(o[e]) * uu[e];
    }
    bf16x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (bf16)o[e];
    *reinterpret_cast<bf16x4*>(C + (size_t)m * N + n) = w;
}

struct SkinnyPlan {
    int n_tiles, kt_per_split, ksplit, rows, rb;
    size_t ws_bytes;
};

template <int RB>
static void skinny_plan_rb(SkinnyPlan& p, int Nrows, int nk) {
    constexpr int kTile = 64 * RB;
    // Units (tiles times K slices) of one round: one per CU, although two fit in most forms.  Half as many K slices halve the partial
    // sums written here and re-read by the consumer (8B decode at 64 tokens, 64-row tiles: qkv 17.7 -> 16.5 us, o 14.8 -> 12.0 us; a
    // target of 128 or 192 units is slower again, 384 and more as well).
    constexpr int kUnits = 256;
    p.rb = RB;
    p.n_tiles = (Nrows + kTile - 1) / kTile;
    int target = kUnits / p.n_tiles;              // aim at one round
    if (target < 1) target = 1;
    p.kt_per_split = (nk + target - 1) / target;
    const int min_kt = nk < 4 * RB ? nk : 4 * RB; // keep the ring worth filling
    if (p.kt_per_split < min_kt) p.kt_per_split = min_kt;
    p.ksplit = (nk + p.kt_per_split - 1) / p.kt_per_split;
    // A grid a little short of a multiple of the units leaves some CUs idle for the whole kernel, or for its last round.
    // Narrower tiles (down to half of the rows, in steps of 8) bring the count up to the multiple; narrower than that, the
    // activations would be re-read by too many tiles.  (88 of 128 rows: 7B gate/up 172 -> 251 workgroups, 30.8 -> 29.6 us at
    // 12 rows, 39.2 -> 37.5 at 64.)  Half against three quarters of the rows, cold weights, time ratios of products whose plan
    // that changes: long streams (26) 0.77 at 8 rows, 0.79 at 32, 0.87 at 64.  Short streams in several rounds (16) 0.95 to 0.97 at 6 rows,
    // 0.94 at 24, 0.91 to 0.94 at 64; in a single round (44) 1.005 up to 24 rows (0.1 us; the worst 8704 x 512 9.7 -> 10.0), 0.96 to 0.97
    // at 64.  (The tiles do not look at the rows, so that a row's sums are the same in every batch of up to 64.)
    p.rows = kTile;
    const int total = p.n_tiles * p.ksplit;
    const int rounds = (total + kUnits - 1) / kUnits;
    const int want_tiles = rounds * kUnits / p.ksplit;
    if (want_tiles > p.n_tiles) {
        const int r = ((Nrows + want_tiles - 1) / want_tiles + 7) / 8 * 8;
        if (r >= kTile / 2 && r < kTile) {
            p.rows = r;
            p.n_tiles = (Nrows + r - 1) / r;
        }
    }
}

static SkinnyPlan skinny_plan(int M, int N, int K, int mode) {
    SkinnyPlan p;
    const int Nrows = (mode == 2) ? 2 * N : N;
    const int nk = (K + kBK - 1) / kBK;
    const bool stream = (size_t)Nrows * K * sizeof(bf16) >= kSkStreamBytes;
    if (stream) skinny_plan_rb<2>(p, Nrows, nk);
    else skinny_plan_rb<1>(p, Nrows, nk);
    p.ws_bytes = (size_t)p.ksplit * M * Nrows * sizeof(float);
    return p;
}

constexpr int kSkMaxM = 64;
static bool skinny_ok(int M, int N, int K) {
    return M >= 1 && M <= kSkMaxM && K % 8 == 0 && N % 4 == 0 &&
           // problems with a K tail needed no scratch before: none whose sums exceed what callers can hold is taken
           (K % kBK == 0 || (uint64_t)M * 2 * N * sizeof(float) <= kMidMaxPartial) &&
           (uint64_t)2 * N * K < 0x7fffffffull;          // 32-bit byte offsets into the weights (2N rows in gate/up mode)
}

// Short K tails as single products stay with the 64x128 kernel: the decode kernel needs a second launch for the fold and the
// epilogue.  Plain epilogue 6.4 -> 8.5 us at K = 8 to 88, 8.1 and 8.6 at 168, 9.8 and 9.8 at 216; with the residual, whose
// loads grow with the rows in the 64x128 kernel's epilogue, 6.7 -> 9.0 (one row, K = 24), 8.4 and 9.0 (3 rows, 104), 9.9 and
// 8.9 (12 rows, 40), 16.5 and 9 (45 rows).  Gate/up writes its result itself and is never slower.  (In run_layers
// the next step folds the sums, so there it is one launch either way: launch_gemm_partial.)
static bool short_tail(int mode, int M, int K) {
    return K % kBK != 0 && ((mode == 0 && K < 192) || (mode == 1 && M <= 8 && K < 128));
}

size_t gemm_workspace_bytes(int mode, int M, int N, int K) {
    if (skinny_ok(M, N, K)) return short_tail(mode, M, K) ? 0 : skinny_plan(M, N, K, mode).ws_bytes;
    MidPlan p;
    if (mid_takes(mode, M, N, K, kMidMaxPartial, p)) {
        // Up to 256 rows a problem whose output, as one range's sums, is larger than the static scratch is reported with
        // that size, although its K is never cut: the interface promises that such a problem is refused there.
        const size_t one = (size_t)M * ((mode == 2) ? 2 * N : N) * sizeof(float);
        return M <= 256 && one > kMidMaxPartial ? one : p.ws_bytes;
    }
    if (big_ok(M, N, K)) return big_plan(mode, M, N, K).ws_bytes;
    return 0;
}

// What an instance sets aside for a problem.  It is part of bz_query_sizes, which callers keep workspaces by, so it is not
// what the plans would like best: partial sums of up to 256 rows over as many ranges of K as tiles of 64 (long streams:
// 128) weight rows and blocks of 128 rows leave compute units for, and the large tiles' beyond.  run_layers hands the plans
// of a batch the largest of its four projections' (13B output projection, 200 rows: 7.8 MB of sums, its own share 3.9);
// by the time model that costs 174 of the 30 000 plans of five decoder shapes between 65 and 2048 rows more than 1 %, 3.7 % at most
// (13B at 193 rows).
size_t gemm_instance_bytes(int mode, int M, int N, int K) {
    if (M > 256 || K % kBK) return big_ok(M, N, K) ? big_plan(mode, M, N, K).ws_bytes : 0;
    if (M <= kSkMaxM) return skinny_ok(M, N, K) ? skinny_plan(M, N, K, mode).ws_bytes : 0;
    if (!big_ok(M, N, K)) return 0;
    const int Nrows = (mode == 2) ? 2 * N : N, nk = K / kBK;
    const int rb = (size_t)Nrows * K * sizeof(bf16) >= kSkStreamBytes ? 2 : 1;
    const int tiles = (Nrows + 64 * rb - 1) / (64 * rb);
    int ranges = 256 / ((M + 127) / 128) / tiles;
    if (ranges < 1) ranges = 1;
    int per = (nk + ranges - 1) / ranges;
    const int least = nk < 4 * rb ? nk : 4 * rb;
    if (per < least) per = least;
    return (size_t)((nk + per - 1) / per) * M * Nrows * sizeof(float);
}

static bool skinny_applies(int mode, int M, int N, int K, const float* ws, size_t ws_bytes) {
    return skinny_ok(M, N, K) && ws != nullptr && ws_bytes >= skinny_plan(M, N, K, mode).ws_bytes;
}

struct SkinnyArgs {
    const bf16* a; const bf16* w; float* ws; bf16* direct;
    int M, Nrows, K, n_tiles, kt_per_split, rows;
};

template <bool GU, bool NT, int RB, int TB, int ST, bool TAIL>
static void skinny_launch(dim3 grid, hipStream_t st, const SkinnyArgs& g) {
    constexpr int lds = SkCfg<RB, TB, ST>::kLds;
    static LdsLimit limit;               // per instantiation: the LDS limit is a per-function setting
    (void)limit.raise(reinterpret_cast<const void*>(gemm_skinny_kernel<GU, NT, RB, TB, ST, TAIL>), lds);
    hipLaunchKernelGGL((gemm_skinny_kernel<GU, NT, RB, TB, ST, TAIL>), grid, dim3(256), lds, st, g.a, g.w, g.ws, g.direct, g.M,
                       g.Nrows, g.K, g.n_tiles, g.kt_per_split, g.rows);
}

template <bool GU, bool NT, int RB, int TB, int ST>
static void skinny_go(dim3 grid, hipStream_t st, const SkinnyArgs& g) {
    if (g.K % kBK) skinny_launch<GU, NT, RB, TB, ST, true>(grid, st, g);
    else skinny_launch<GU, NT, RB, TB, ST, false>(grid, st, g);
}

template <bool GU>
static void skinny_stream(dim3 grid, hipStream_t st, const SkinnyArgs& g) {
    if (g.M <= 32) skinny_go<GU, true, 2, 1, 4>(grid, st, g);
    else if (grid.x > 256) skinny_go<GU, true, 2, 2, 3>(grid, st, g);
    else skinny_go<GU, true, 2, 2, 4>(grid, st, g);
}

// Split-K partial sums only: partial[ksplit][M][Nrows] (Nrows = 2N in SwiGLU mode).  The caller
// folds the slices in slice order, either with gemm_partial_epilogue or fused into the next kernel.
// `c` (gate/up mode only): where the activation goes when one k-slice covers K; then the return value is 0
// and no partial sums are written.
static int launch_skinny_partial(int mode, const bf16* a, const bf16* w, bf16* c, int M, int N, int K, float* ws,
                                 hipStream_t st) {
    const SkinnyPlan p = skinny_plan(M, N, K, mode);
    const int Nrows = (mode == 2) ? 2 * N : N;
    const dim3 grid(p.n_tiles * p.ksplit);
    bf16* direct = (mode == 2 && p.ksplit == 1) ? c : nullptr;
    const SkinnyArgs args{a, w, ws, direct, M, Nrows, K, p.n_tiles, p.kt_per_split, p.rows};
    const bool gu = mode == 2;
    if (p.rb == 2) {
        if (gu) skinny_stream<true>(grid, st, args); else skinny_stream<false>(grid, st, args);
    } else {
        if (gu) skinny_go<true, false, 1, 2, 4>(grid, st, args); else skinny_go<false, false, 1, 2, 4>(grid, st, args);
    }
    if (direct) return 0;
    return p.ksplit;
}

int launch_gemm_partial(int mode, const act_t* a, const bf16* w, int M, int N, int K, float* ws, size_t ws_bytes,
                        hipStream_t st) {
    if (M <= 0 || N <= 0) return 0;
    if (skinny_applies(mode, M, N, K, ws, ws_bytes)) return launch_skinny_partial(mode, a, w, nullptr, M, N, K, ws, st);
    MidPlan p;
    if (ws == nullptr || !mid_takes(mode, M, N, K, ws_bytes, p) || p.ksplit == 1) return 0;
    return launch_mid(mode, p, a, w, nullptr, nullptr, M, N, K, ws, st) ? p.ksplit : 0;
}

// Adds the slices of `ws` in slice order and applies the epilogue.
template <int MODE>
static void launch_partial_epilogue(const float* ws, const bf16* r, bf16* c, int M, int N, int ksplit, hipStream_t st) {
    const int threads = M * (N >> 2);
    hipLaunchKernelGGL(gemm_partial_epilogue<MODE>, dim3((threads + 255) / 256), dim3(256), 0, st, ws, r, c, M, N,
                       (MODE == 2) ? 2 * N : N, ksplit);
}

template <int MODE>
static void launch_skinny(const bf16* a, const bf16* w, const bf16* r, bf16* c, int M, int N, int K, float* ws,
                          hipStream_t st) {
    const int ksplit = launch_skinny_partial(MODE, a, w, c, M, N, K, ws, st);
    if (ksplit == 0) return;                          // the kernel wrote the result itself
    launch_partial_epilogue<MODE>(ws, r, c, M, N, ksplit, st);
}

// false: not a problem of the mid-sized kernel (or no LDS for it).
template <int MODE>
static bool launch_mid_whole(const bf16* a, const bf16* w, const bf16* r, bf16* c, int M, int N, int K, float* ws,
                             size_t ws_bytes, hipStream_t st) {
    MidPlan p;
    if (!mid_takes(MODE, M, N, K, ws == nullptr ? 0 : ws_bytes, p)) return false;
    if (!launch_mid(MODE, p, a, w, r, c, M, N, K, ws, st)) return false;
    if (p.ksplit > 1) launch_partial_epilogue<MODE>(ws, r, c, M, N, p.ksplit, st);
    return true;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int MODE>
static void launch_cfg(const bf16* a, const bf16* w, const bf16* r, bf16* c, int M, int N, int K, hipStream_t st) {
    constexpr int OUT_BN = (MODE == 2) ? BN / 2 : BN;
    constexpr int LDS = gemm_lds_bytes<BM, BN>();
    auto kern = gemm_kernel<BM, BN, WAVES_M, WAVES_N, MODE>;
    static LdsLimit limit;             // one per instantiation
    (void)limit.raise(reinterpret_cast<const void*>(kern), LDS);
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + OUT_BN - 1) / OUT_BN;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(WAVES_M * WAVES_N * 64), LDS, st, a, w, r, c, M, N, K,
                       tiles_m, tiles_n);
}

template <int MODE>
static void launch_mode(const bf16* a, const bf16* w, const bf16* r, bf16* c, int M, int N, int K, float* ws,
                        size_t ws_bytes, hipStream_t st) {
    // The kernel and its tiling are a function of the problem's shape and the scratch, and that in run_layers one of the model
    // and the rows: a layer's result never depends on which range of layers a call covers, or on the instance.
    if (skinny_applies(MODE, M, N, K, ws, ws_bytes) && !short_tail(MODE, M, K)) {
        launch_skinny<MODE>(a, w, r, c, M, N, K, ws, st);
    } else if (M <= 64) {
        launch_cfg<64, 128, 2, 2, MODE>(a, w, r, c, M, N, K, st);
    } else if (launch_mid_whole<MODE>(a, w, r, c, M, N, K, ws, ws_bytes, st)) {
        return;
    } else if (big_ok(M, N, K) && big_available<MODE>()) {
        launch_big<MODE>(a, w, r, c, M, N, K, ws, ws_bytes, st);
    } else {
        launch_cfg<128, 128, 2, 2, MODE>(a, w, r, c, M, N, K, st);
    }
}

// What launch_mode does with `room` bytes of scratch, where every kernel gets its LDS.
void gemm_plan(int mode, int M, int N, int K, size_t room, bz_gemm_plan* out) {
    *out = bz_gemm_plan{};
    if (M <= 0 || N <= 0) return;
    const int Nrows = (mode == 2) ? 2 * N : N;
    MidPlan mid;
    if (room > 0 && skinny_ok(M, N, K) && skinny_plan(M, N, K, mode).ws_bytes <= room && !short_tail(mode, M, K)) {
        const SkinnyPlan p = skinny_plan(M, N, K, mode);
        *out = bz_gemm_plan{BZ_GEMM_DECODE, 64, p.rows, 1, p.n_tiles, 0, p.ksplit, p.ws_bytes};
    } else if (M > 64 && mid_takes(mode, M, N, K, room, mid)) {
        const MidTile& t = kMidTiles[mid.tile];
        *out = bz_gemm_plan{BZ_GEMM_MID, t.wt * t.nbt * 16, (4 / t.wt) * t.nbf * 16, mid.m_tiles, mid.n_tiles, 0, mid.ksplit,
                            mid.ws_bytes};
    } else if (M > 64 && big_ok(M, N, K)) {
        const BigPlan p = big_plan(mode, M, N, K);
        const bool split = p.tail > 0 && p.ws_bytes <= room;
        *out = bz_gemm_plan{BZ_GEMM_LARGE, 256, 256, p.tiles_m, p.tiles_n, split ? p.n_dp : p.tiles_m * p.tiles_n,
                            split ? p.splits : 1, split ? p.ws_bytes : 0};
    } else {
        const int bm = M <= 64 ? 64 : 128;
        *out = bz_gemm_plan{BZ_GEMM_SMALL, bm, 128, (M + bm - 1) / bm, (Nrows + 127) / 128, 0, 1, 0};
    }
}

void launch_gemm(int mode, const act_t* a, const bf16* w, const act_t* r, act_t* c, int M, int N, int K,
                 float* ws, size_t ws_bytes, hipStream_t st) {
    if (M <= 0 || N <= 0) return;
    switch (mode) {
        case 0: launch_mode<0>(a, w, r, c, M, N, K, ws, ws_bytes, st); break;
        case 1: launch_mode<1>(a, w, r, c, M, N, K, ws, ws_bytes, st); break;
        default: launch_mode<2>(a, w, r, c, M, N, K, ws, ws_bytes, st); break;
    }
}

#else  // BZ_FP32_DEBUG: one thread per output element, fp32 FMA chain in k order

template <int MODE>
__global__ __launch_bounds__(256) void gemm_naive_kernel(const float* __restrict__ A, const bf16* __restrict__ W,
                                                         const float* R, float* C, int M, int N, int K) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)M * N) return;
    const int m = (int)(idx / N), n = (int)(idx % N);
    const float* a = A + (size_t)m * K;
    if (MODE == 2) {
        const bf16* wg = W + (size_t)n * K;
        const bf16* wu = W + (size_t)(N + n) * K;
        float g = 0.f, u = 0.f;
        for (int k = 0; k < K; ++k) {
            g = fmaf(a[k], (float)wg[k], g);
            u = fmaf(a[k], (float)wu[k], u);
        }
        C[idx] = g / (1.0f + expf(-g)) * u;
    } else {
        const bf16* w = W + (size_t)n * K;
        float s = 0.f;
        for (int k = 0; k < K; ++k) s = fmaf(a[k], (float)w[k], s);
        if (MODE == 1) s += R[idx];
        C[idx] = s;
    }
}

size_t gemm_workspace_bytes(int, int, int, int) { return 0; }
size_t gemm_instance_bytes(int, int, int, int) { return 0; }
void gemm_plan(int, int, int, int, size_t, bz_gemm_plan* out) { *out = bz_gemm_plan{}; }
int launch_gemm_partial(int, const act_t*, const bf16*, int, int, int, float*, size_t, hipStream_t) { return 0; }

void launch_gemm(int mode, const act_t* a, const bf16* w, const act_t* r, act_t* c, int M, int N, int K,
                 float*, size_t, hipStream_t st) {
    if (M <= 0 || N <= 0) return;
    const size_t total = (size_t)M * N;
    const dim3 grid((unsigned)((total + 255) / 256));
    switch (mode) {
        case 0: hipLaunchKernelGGL(gemm_naive_kernel<0>, grid, dim3(256), 0, st, a, w, r, c, M, N, K); break;
        case 1: hipLaunchKernelGGL(gemm_naive_kernel<1>, grid, dim3(256), 0, st, a, w, r, c, M, N, K); break;
        default: hipLaunchKernelGGL(gemm_naive_kernel<2>, grid, dim3(256), 0, st, a, w, r, c, M, N, K); break;
    }
}

#endif

}  // namespace bz
