// Projections of a batch of one to four rows (an answer being written, the shortest prompts), the norm in front of them and the
// residual or SwiGLU behind them included: a decoder layer is the attention and four of these launches, and neither partial
// sums nor normalised rows travel through memory.  (From 5 rows on: two norms, four products cut over K, their sums folded by
// the next kernel, and a combine launch.)
//
// Bound: the weights, read once.  One workgroup per CU takes a run of weight rows; its 8 waves share out K, each streaming its
// part of 16 to 32 rows per step, one cache line per row, through a ring of its own in LDS, with no barrier but one per tile:
// that keeps 32 to 96 KiB in flight per CU.  Tried before: the weights straight into registers in the matrix instruction's
// operand order (16 rows of 64 bytes per load): 8B-GQA gate/up 48 us against 38.6, a lane's neighbours being in other lines.
// The norm hides behind the first weights: its rows are requested first, and it runs while the ring fills.
//
// Measured (one row, 8B-GQA / 7B / 13B / 70B, us): QKV with the norm 10.6 / 18 / 27 / 28.5, output projection with the combine
// 8.9 / 10 / 14 / 29.6, gate/up with the norm 37.7 (6.2 TB/s) / 31 / 46 / 145 (6.5 TB/s), down 19.6 / 16.5 / 24.4 / 73.5.  As
// separate kernels at 8B-GQA: norms 4.2 each, QKV 9.8 to 12, output projection 7.6, combine 4.5, gate/up 38, down 20.  One layer,
// before and after: 8B-GQA one row 101 -> 88, four 101 -> 94; 70B one 307 -> 296, four 310 -> 308; 13B one 139 -> 130, three
// 148 -> 143; 7B one 105 -> 93.  Beyond four rows the rows' part of the norm, done by every workgroup, outweighs the launches
// saved on some shapes (8B-GQA five 105 -> 103, eight 110.5 -> 110; 7B 112 -> 114 and 125 -> 128).
#include <type_traits>

#include "common.h"
#include "few_rows.h"

namespace bz {

#ifndef BZ_FP32_DEBUG

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kFewWaves = kFewThreads / kWave;
constexpr int kFewK = 64;                    // columns of a step: one cache line of a weight row
constexpr int kFewPad = 64;                  // bytes between the rows in LDS, so that their reads of one step spread over the banks
constexpr int kFewLds = 160 * 1024;

// Where the rows come from: memory, step by step with the weights; the residual stream, normalised; the partial results of
// the decode attention, combined.
enum { kRows = 0, kNorm = 1, kCombine = 2 };

// A tile is NR groups of 8 weight rows, multiplied in NB blocks of 16.
// LDS: [2][waves][NB * 4][M] f32x4 of a tile's sums, the prepared rows, then every wave's ring of D slots
template <int SRC, int NR> struct FewCfg {
    static constexpr int NB = (NR + 1) / 2;
    static constexpr int kLoads = NR + (SRC == kRows ? 1 : 0);       // of 1 KiB per step
    static constexpr int kSlot = kLoads * 1024;
    __host__ __device__ static constexpr int red_bytes(int M) { return 2 * kFewWaves * NB * 4 * M * 16; }
    __host__ __device__ static constexpr int ring_at(int M, int K) {
        return (red_bytes(M) + (SRC == kRows ? 0 : M * (K * 2 + kFewPad)) + 1023) / 1024 * 1024;
    }
};

__device__ __forceinline__ int few_swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }
__device__ __forceinline__ constexpr int few_vmcnt(int n) { return ((n >> 4) << 14) | 0x0f70 | (n & 15); }

// Sum over the wave, in lane 63: shifts inside rows of 16 lanes, then broadcasts of the rows' last lanes.  The norm is a chain of
// dependent steps here, and a shuffle is a trip through LDS (the smallest session 511 -> 498 us).
__device__ __forceinline__ float last_lane_sum(float v) {
    auto moved = [](float x, auto ctrl, auto rows) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                     decltype(rows)::value, 0xf, false));
    };
    using All = std::integral_constant<int, 0xf>;
    v += moved(v, std::integral_constant<int, 0x111>(), All());                                  // row_shr:1, 2, 4, 8
    v += moved(v, std::integral_constant<int, 0x112>(), All());
    v += moved(v, std::integral_constant<int, 0x114>(), All());
    v += moved(v, std::integral_constant<int, 0x118>(), All());
    v += moved(v, std::integral_constant<int, 0x142>(), std::integral_constant<int, 0xa>());     // row_bcast:15
    v += moved(v, std::integral_constant<int, 0x143>(), std::integral_constant<int, 0xc>());     // row_bcast:31
    return v;
}

struct FewArgs {
    const bf16* x;           // rows; kNorm: the residual stream
    const bf16* gain;        // kNorm
    float eps;
    const bf16* w;
    const bf16* r;           // EPI 1: residual (may be c)
    bf16* c;
    int M, N, K;
    int units, per_wg;       // groups of 4 weight rows (EPI 2: of 4 features), all and per workgroup
    const float* partial;    // kCombine: of row m, head h, chunk j at ((m * heads + h) * chunks + j) * (d + 2)
    const int32_t* kv_before;
    int d, chunks;
};

// EPI 0: c = the product; 1: c = r + product; 2: the weights are N gate rows, then N up rows, c = silu(gate) * up.
// TAIL: K is no multiple of 64 (but of 8).  D: steps in flight per wave.  SLOTS: kNorm: 8-element vectors of the rows that a
// thread normalises; kCombine: chunks.  TOK (kCombine): rows.
template <int SRC, int EPI, int NR, bool TAIL, int D, int SLOTS, int TOK>
__global__ __launch_bounds__(kFewThreads, 2) void gemm_few_kernel(const FewArgs a) {
    using Cfg = FewCfg<SRC, NR>;
    constexpr int NW = kFewWaves, NB = Cfg::NB, P = Cfg::kLoads, kSlot = Cfg::kSlot;
    static_assert(EPI != 2 || NR == 2, "a block of gate and up rows");
    constexpr int kTile = EPI == 2 ? 8 : NR * 8;                      // rows (EPI 2: features)
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const int M = a.M, N = a.N, K = a.K;
    f32x4* red = reinterpret_cast<f32x4*>(smem_raw);
    const int xs = Cfg::red_bytes(M);                                 // byte offset of the prepared rows
    const int pitch = K * 2 + kFewPad;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, g = lane >> 4;                         // weight row / token, and 8-element group of an MFMA's 32 columns
    const int tok = col < M ? col : M - 1;
    const int steps = (K + kFewK - 1) / kFewK;
    const int s0 = steps * wave / NW, count = steps * (wave + 1) / NW - s0;      // this wave's steps of a tile
    const int n0 = blockIdx.x * a.per_wg * 4;                         // this workgroup's rows (features) n0 .. n1 - 1
    const int n1 = n0 + a.per_wg * 4 < N ? n0 + a.per_wg * 4 : N;
    const int ntiles = EPI == 1 ? 1 : (n1 - n0 + kTile - 1) / kTile;

    // what the rows are made of is requested before the weights (loads complete in order)
    const int nvec = K >> 3;
    const bool wide = nvec > kFewThreads;                             // two vectors per thread and row
    bf16x8 xv[SRC == kNorm ? SLOTS : 1], gv[2];
    if (SRC == kNorm) {
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
            int m = wide ? q >> 1 : q;
            if (m > M - 1) m = M - 1;
            int i = tid + (wide ? (q & 1) * kFewThreads : 0);
            if (i > nvec - 1) i = nvec - 1;
            xv[q] = *reinterpret_cast<const bf16x8*>(a.x + (size_t)(uint32_t)(m * K + i * 8));
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            int i = tid + c * kFewThreads;
            if (i > nvec - 1) i = nvec - 1;
            gv[c] = *reinterpret_cast<const bf16x8*>(a.gain + i * 8);
        }
    }
    // a lane combines 8 columns of its wave's share of K
    const int c0 = s0 * kFewK, c1 = c0 + count * kFewK;
    int nch[SRC == kCombine ? TOK : 1];
    float2 ov[SRC == kCombine ? TOK : 1][SRC == kCombine ? SLOTS : 1][4], ml[SRC == kCombine ? TOK : 1][SRC == kCombine ? SLOTS : 1];
    const int PS = a.d + 2;
    auto load_parts = [&](int k) {                                    // columns k .. k + 7; past the share the last ones
        const int kc = k < c1 ? k : c1 > 8 ? c1 - 8 : 0;
        const int head = kc / a.d, dd = kc - head * a.d;
#pragma unroll
        for (int m = 0; m < TOK; ++m)
#pragma unroll
            for (int j = 0; j < SLOTS; ++j) {
                const float* p = a.partial + ((size_t)(m * (K / a.d) + head) * a.chunks + (j < a.chunks ? j : a.chunks - 1)) * PS;
#pragma unroll
                for (int e = 0; e < 4; ++e) ov[m][j][e] = *reinterpret_cast<const float2*>(p + dd + 2 * e);
                ml[m][j] = *reinterpret_cast<const float2*>(p + a.d);
            }
    };
    if (SRC == kCombine) {
#pragma unroll
        for (int m = 0; m < TOK; ++m) nch[m] = a.kv_before[m] / kDecodeChunk + 1;
        load_parts(c0 + lane * 8);
    }
    // block j of tile t is finished by wave (t * NB + j) % NW
    auto block_of = [&](int t) { return (wave - t * NB) & (NW - 1); };
    bf16x4 rv;
    if (EPI == 1) {                                                   // one tile only: N is the hidden size, 32 rows per workgroup at most
        int n = n0 + wave * 16 + 4 * g;
        if (n > N - 4) n = N - 4;                                     // value unused
        rv = *reinterpret_cast<const bf16x4*>(a.r + (size_t)tok * N + n);
    }
    __builtin_amdgcn_sched_barrier(0);

    // A step's loads of 1 KiB: NR times 8 weight rows of one cache line each, and (kRows) the line of every row.  The 16-byte
    // pieces of a row are fetched in an order that depends on the row, so that the operand reads hit different banks.
    const int lr = lane >> 3;
    const uint32_t piece[2] = {(uint32_t)((lane & 7) ^ few_swz(lr)) * 8, (uint32_t)((lane & 7) ^ few_swz(lr + 8)) * 8};
    const uint32_t wbytes = (EPI == 2 ? 2u : 1u) * (uint32_t)N * (uint32_t)K * 2u, xbytes = (uint32_t)M * (uint32_t)K * 2u;
    unsigned char* ring = smem_raw + Cfg::ring_at(M, K) + wave * (D * kSlot);
    const uint32_t xrow = (uint32_t)(lr < M ? lr : M - 1) * (uint32_t)K;
    auto column = [&](int s, uint32_t piece) {                        // pieces past K re-read the row's last one
        uint32_t k = (uint32_t)s * kFewK + piece;
        if (TAIL && k > (uint32_t)K - 8) k = (uint32_t)K - 8;
        return k;
    };
    // A workgroup starts its walk over the columns where its number says and wraps around, so that not all of them ask the
    // same memory channels at a time (8B-GQA down projection 21.1 -> 20.0 us).
    const int rot = count ? (int)(blockIdx.x % (unsigned)count) : 0;
    auto step_of = [&](int i) { return s0 + (i + rot >= count ? i + rot - count : i + rot); };
    // Past the last step the requests go on through empty resources, which costs no memory traffic: every step has the same
    // number of loads behind it, and the waits are constants.  So do rows past the workgroup's last one, by an offset past
    // every end.  (All of an offset is in its vector part: the range check of an empty resource must not wrap.)
    const int total = count * ntiles;
    int issued = 0, it = 0, is = 0, islot = 0;                        // tile, step and slot of the next request
    auto issue = [&] {
        const bool on = issued < total;
        ++issued;
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, on ? (int)wbytes : 0, 0x00020000);
        const int s = step_of(is);
        unsigned char* dst = ring + islot * kSlot;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const uint32_t r = n0 + it * kTile + (EPI == 2 ? 0 : j * 8) + lr;
            const uint32_t k = column(s, piece[j & 1]);
            const uint32_t o = (int)r < n1 ? ((EPI == 2 && j ? N + r : r) * (uint32_t)K + k) * 2u : 0xfffffff0u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lptr_t)(dst + j * 1024), 16, (int)o, 0, 0, 2);
        }
        if (SRC == kRows) {
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, on ? (int)xbytes : 0, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lptr_t)(dst + NR * 1024), 16, (int)((xrow + column(s, piece[0])) * 2u), 0, 0, 0);
        }
        islot = islot + 1 == D ? 0 : islot + 1;
        if (++is == count) { is = 0; ++it; }
    };
#pragma unroll
    for (int q = 0; q < D; ++q) issue();
    __builtin_amdgcn_sched_barrier(0);

    // Own LDS accesses are done, then everyone's.  Written out, because a fence would wait for the loads into the ring as well.
    auto lds_barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    if (SRC == kNorm) {
        float* ssq = reinterpret_cast<float*>(smem_raw);              // [SLOTS][NW] in the place of the sums
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = fmaf((float)xv[q][e], (float)xv[q][e], ss);
            ss = last_lane_sum(tid + (wide ? (q & 1) * kFewThreads : 0) < nvec ? ss : 0.f);
            if (lane == 63) ssq[q * NW + wave] = ss;
        }
        lds_barrier();
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
            const int m = wide ? q >> 1 : q, i = tid + (wide ? (q & 1) * kFewThreads : 0);
            if (m < M && i < nvec) {
                float tot = 0.f;
                const int q0 = wide ? q & ~1 : q;
#pragma unroll
                for (int w = 0; w < NW; ++w) tot += ssq[q0 * NW + w];
                if (wide)
#pragma unroll
                    for (int w = NW; w < 2 * NW; ++w) tot += ssq[q0 * NW + w];
                const float rstd = 1.0f / sqrtf(tot / (float)K + a.eps);
                const bf16x8 gq = wide && (q & 1) ? gv[1] : gv[0];
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (bf16)(((float)xv[q][e] * rstd) * (float)gq[e]);
                *reinterpret_cast<bf16x8*>(smem_raw + xs + m * pitch + i * 16) = o;
            }
        }
        lds_barrier();
    }
    if (SRC == kCombine) {                                            // as attn_combine_kernel does; a wave needs its own columns only
        for (int k = c0 + lane * 8;; k += kWave * 8) {
#pragma unroll
            for (int m = 0; m < TOK; ++m) {
                float mx = -INFINITY, den = 0.f, num[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < SLOTS; ++j) mx = fmaxf(mx, j < nch[m] ? ml[m][j].x : -INFINITY);
#pragma unroll
                for (int j = 0; j < SLOTS; ++j)
                    if (j < nch[m]) {
                        const float w = exp2f(ml[m][j].x - mx);
                        den = fmaf(ml[m][j].y, w, den);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            num[2 * e] = fmaf(ov[m][j][e].x, w, num[2 * e]);
                            num[2 * e + 1] = fmaf(ov[m][j][e].y, w, num[2 * e + 1]);
                        }
                    }
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (bf16)(num[e] / den);
                if (m < M && k < c1) *reinterpret_cast<bf16x8*>(smem_raw + xs + m * pitch + k * 2) = o;
            }
            if (k - lane * 8 + kWave * 8 >= c1) break;                // wave-uniform
            load_parts(k + kWave * 8);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }

    f32x4 acc[NB];
    const int wat = col * 128, wsw = few_swz(col), xat = SRC == kRows ? NR * 1024 + tok * 128 : xs + tok * pitch, xsw = few_swz(tok);
    int slot = 0;
    for (int t = 0; t < ntiles; ++t) {
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int i = 0; i < count; ++i) {
            const int s = step_of(i);
            // the step has landed; the D - 1 requested after it may be in flight (other loads and stores in between only make
            // the wait stricter)
            __builtin_amdgcn_s_waitcnt(few_vmcnt((D - 1) * P));
            __builtin_amdgcn_sched_barrier(0);
            const unsigned char* st = ring + slot * kSlot;
            bf16x8 w[NB][2], x[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const bool past = TAIL && s * kFewK + ks * 32 + g * 8 >= K;
                if (SRC == kRows) x[ks] = *reinterpret_cast<const bf16x8*>(st + xat + ((ks * 4 + g) ^ xsw) * 16);
                else x[ks] = *reinterpret_cast<const bf16x8*>(smem_raw + xat + (past ? 0 : s * 128 + ks * 64 + g * 16));
                if (past) x[ks] = bf16x8{};
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    // with an odd NR the last block's second half is the slot's last rows again, and not used
                    const int at = NR % 2 && j == NB - 1 ? wat & 0x3ff : wat;
                    w[j][ks] = *reinterpret_cast<const bf16x8*>(st + j * 2048 + at + ((ks * 4 + g) ^ wsw) * 16);
                    if (past) w[j][ks] = bf16x8{};
                }
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);                       // lgkmcnt(0): the slot has been read
            __builtin_amdgcn_sched_barrier(0);
            issue();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j][ks], x[ks], acc[j], 0, 0, 0);
            slot = slot + 1 == D ? 0 : slot + 1;
        }
        // add up the waves' parts of the tile, in wave order
        f32x4* part = red + (t & 1) * (NW * NB * 4 * M);
        if (col < M)
#pragma unroll
            for (int j = 0; j < NB; ++j) part[((wave * NB + j) * 4 + g) * M + col] = acc[j];
        lds_barrier();
        const int jb = block_of(t);
        if (jb < NB && col < M && (EPI != 2 || g < 2)) {
            f32x4 sum = {0.f, 0.f, 0.f, 0.f}, up = sum;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                sum += part[((w * NB + jb) * 4 + g) * M + col];
                if (EPI == 2) up += part[((w * NB + jb) * 4 + g + 2) * M + col];
            }
            const int local = jb * 16 + 4 * g, n = n0 + t * kTile + local;
            if (local < kTile && n < n1) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (EPI == 2) o[e] = (bf16)(silu_fast(sum[e]) * up[e]);
                    else if (EPI == 1) o[e] = (bf16)(sum[e] + (float)rv[e]);
                    else o[e] = (bf16)sum[e];
                }
                *reinterpret_cast<bf16x4*>(a.c + (size_t)col * N + n) = o;
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(few_vmcnt(0));                         // no LDS write may be in flight when the workgroup ends
}

template <int SRC, int EPI, int NR, int D, int SLOTS = 1, int TOK = 1>
static void launch_few_d(const FewArgs& a, hipStream_t st) {
    const int lds = FewCfg<SRC, NR>::ring_at(a.M, a.K) + kFewWaves * D * FewCfg<SRC, NR>::kSlot;
    const bool tail = a.K % kFewK != 0;
    auto kern = tail ? gemm_few_kernel<SRC, EPI, NR, SRC != kCombine, D, SLOTS, TOK> : gemm_few_kernel<SRC, EPI, NR, false, D, SLOTS, TOK>;
    static LdsLimit limit[2];
    (void)limit[tail].raise(reinterpret_cast<const void*>(kern), kFewLds);
    hipLaunchKernelGGL(kern, dim3((a.units + a.per_wg - 1) / a.per_wg), dim3(kFewThreads), lds, st, a);
}

// Steps in flight: as few as keep the stream going, because what is requested first holds back the norm or the combine, whose
// own values are requested before but unpacked after it: with rings of about 128 KiB (8 steps of 16 rows, 5 of 24, 4 of 32) four
// decode steps of the 8B-GQA shape take 1454 us, with 4, 3 and 2 1406, with these 1402, with 2 everywhere 1414.
template <int EPI, int NR, int D>
static void launch_few_norm(const FewArgs& a, hipStream_t st) {
    const int vectors = a.M * few_vectors(a.K);
    if (vectors > 4) launch_few_d<kNorm, EPI, NR, D, 8>(a, st);
    else if (vectors > 2) launch_few_d<kNorm, EPI, NR, D, 4>(a, st);
    else launch_few_d<kNorm, EPI, NR, D, 2>(a, st);
}

template <int NR, int D>
static void launch_few_combine(const FewArgs& a, hipStream_t st) {
    if (a.M == 2) launch_few_d<kCombine, 1, NR, D, 8, 2>(a, st);
    else if (a.chunks <= 8) launch_few_d<kCombine, 1, NR, D, 8, 1>(a, st);
    else launch_few_d<kCombine, 1, NR, D, 16, 1>(a, st);
}

// Weight rows per workgroup (one per CU), in groups of 4, and the row groups of 8 of a tile: as many as they are, up to four;
// where they are more, tiles of about the same size.
static int few_cut(FewArgs& a) {
    a.units = (a.N + 3) / 4;
    a.per_wg = (a.units + 255) / 256;
    const int tiles = (a.per_wg + 7) / 8, rows = (a.per_wg + tiles - 1) / tiles * 4;
    return rows <= 16 ? 2 : rows <= 24 ? 3 : 4;
}

// Whether the output projection combines the chunks itself: every workgroup reads all partial results then, which is cheap for
// up to 16 chunks altogether (one row of 4 or 5 chunks: 13.1 -> 10.5 us at 8B-GQA, two rows 13.5 -> 12.3).
bool few_combines(const BatchView& bv, int qd) {
    return bv.n_decode == bv.T && bv.B == bv.T && bv.T <= 2 && bv.n_decode_work > bv.n_decode && bv.T * bv.decode_chunks <= 16 && qd <= 8192;
}

void launch_few_out(const float* partial, const BatchView& bv, const KvView& kv, const bf16* w, act_t* x, int H, int qd, hipStream_t st) {
    FewArgs a{nullptr, nullptr, 0.f, w, x, x, bv.T, H, qd, 0, 0, partial, bv.kv_before, kv.d, bv.decode_chunks};
    switch (few_cut(a)) {
        case 2: launch_few_combine<2, 3>(a, st); break;
        case 3: launch_few_combine<3, 2>(a, st); break;
        default: launch_few_combine<4, 2>(a, st);
    }
}

void launch_few(int mode, const act_t* x, const bf16* gain, float eps, const bf16* w, const act_t* r, act_t* c, int M, int N,
                int K, hipStream_t st) {
    FewArgs a{x, gain, eps, w, r, c, M, N, K, 0, 0, nullptr, nullptr, 0, 0};
    const int nr = few_cut(a);
    // Up to 1024 columns a wave has two steps of a tile at most: two slots do (hidden 256: 3.80 / 3.88 us with two / three for QKV, 3.88 /
    // 4.02 for gate/up; 1024: 3.84 / 4.07 and 5.35 / 5.57, four rows 5.10 / 5.28 and 6.64 / 6.69).  From 2048 on they win nothing (16-row tiles of
    // QKV 4.77 / 4.76) and lose on long streams (8B-GQA gate/up 38.7 / 38.4).
    const bool small = K <= 1024 && nr == 2;
    if (mode == 2) {
        if (small) launch_few_norm<2, 2, 2>(a, st);
        else launch_few_norm<2, 2, 3>(a, st);
    } else if (mode == 0) {
        if (small) launch_few_norm<0, 2, 2>(a, st);
        else if (nr == 2) launch_few_norm<0, 2, 3>(a, st);
        else if (nr == 3) launch_few_norm<0, 3, 3>(a, st);
        else launch_few_norm<0, 4, 2>(a, st);
    } else {
        if (nr == 2) launch_few_d<kRows, 1, 2, 2>(a, st);
        else if (nr == 3) launch_few_d<kRows, 1, 3, 3>(a, st);
        else launch_few_d<kRows, 1, 4, 2>(a, st);
    }
}

#else

bool few_combines(const BatchView&, int) { return false; }
void launch_few_out(const float*, const BatchView&, const KvView&, const bf16*, act_t*, int, int, hipStream_t) {}
void launch_few(int, const act_t*, const bf16*, float, const bf16*, const act_t*, act_t*, int, int, int, hipStream_t) {}

#endif

}  // namespace bz
