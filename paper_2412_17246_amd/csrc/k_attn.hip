// Causal attention over the KV cache: a tiled MFMA kernel for sequences with several new tokens
// (prefill) and a split-KV kernel plus fixed-order combine for sequences with one (decode).
//
// Cache layout per (layer, slot, kv head): blocks of 32 positions, K piece-major (k_elem_offset), V
// in pieces of 8 positions (v_elem_offset): both are the row-operand order of the 32x32x16 MFMA.
// Query head h reads kv head h / (Hq/Hkv).  A query at absolute position p sees keys 0..p.  Scores
// are scaled by 1/sqrt(d); softmax is evaluated in base 2 (scores pre-multiplied by log2 e).
//
// V is multiplied by probability 0 (not skipped) at masked positions of a partly visible block, so
// cache memory must hold finite values everywhere: the arena is cleared when an instance is created
// and only finite values are ever written by the kernels.
#include "common.h"

namespace bz {

// Loads of cache contents that are read once per step (decode attention): non-temporal, so that the
// stream does not push through the caches what nobody will read again; on this chip a streaming read
// of that kind runs about a quarter faster than a default one.
template <class T>
__device__ __forceinline__ T stream_load(const T* ptr) { return __builtin_nontemporal_load(ptr); }

constexpr float kLog2e = 1.4426950408889634f;

#ifndef BZ_FP32_DEBUG
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// 2^x by the hardware instruction alone (results below the normal range flush to zero, which is
// what a softmax weight that small should be anyway)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ---------------------------------------------------------------------------------------------
// Prefill.  One workgroup = 128 query rows of one (sequence, head); each of its 4 waves owns 32
// rows.  The wave computes S^T = K * Q^T with 32x32x16 MFMAs, so that a lane (and its partner
// lane + 32) holds all scores of ONE query row: row max / sum need a single cross-lane exchange
// and the running rescale of O^T is a per-lane scalar.  P^T feeds the second MFMA (O^T = V^T *
// P^T) straight from registers: the accumulator layout of S^T is a permutation of the B-operand
// layout along the contraction index, and the V cache stores its pieces in that permuted order.
//
// A KV tile is 64 positions = two cache blocks of K and two of V, each block contiguous in the
// cache in exactly the order the MFMAs read it, so a tile is moved global -> LDS by the DMA path
// (no registers), double-buffered: tile i+1 is in flight while tile i is multiplied.
//
// SETS = 2: a workgroup takes 64 rows, two waves along them and two along the keys: the second pair takes every other KV
// tile through LDS buffers of its own, and the two parts of a row's result are merged through LDS at the end.  A wave's
// tiles are a serial chain of 1.4 us each with one wave per SIMD, and a second wave on the SIMD shortens nothing (the
// vector and the matrix work of all its waves add up), so a grid that leaves CUs idle gains by halving the chains.
// ---------------------------------------------------------------------------------------------
// A lane's query fragments qf[ks] hold dims 16 ks + 8 lh + 0..7 of one row, so both halves of a rotation pair (j, j + D/2)
// are in the same lane: the query is rotated as it is loaded.  ROTATED: it already is (launch_kv_append).
template <int D, bool ROTATED>
__device__ __forceinline__ void load_query(const bf16* q, const float* cs, bf16x8 (&qf)[D / 16], int lh) {
    constexpr int H = D / 32;                                 // fragments per half of the head
    if (ROTATED) {
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(q + ks * 16 + lh * 8);
        return;
    }
#pragma unroll
    for (int ks = 0; ks < H; ++ks) {
        const int j = ks * 16 + lh * 8;
        float lo[8], hi[8];
        load8(q + j, lo);
        load8(q + D / 2 + j, hi);
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const float4 v = *reinterpret_cast<const float4*>(cs + 2 * (j + e));
            qf[ks][e] = (bf16)(lo[e] * v.x - hi[e] * v.y);
            qf[ks + H][e] = (bf16)(hi[e] * v.x + lo[e] * v.y);
            qf[ks][e + 1] = (bf16)(lo[e + 1] * v.z - hi[e + 1] * v.w);
            qf[ks + H][e + 1] = (bf16)(hi[e + 1] * v.z + lo[e + 1] * v.w);
        }
    }
}

template <int D, bool ROTATED, int SETS>
__global__ __launch_bounds__(256, 2) void attn_prefill_kernel(const bf16* __restrict__ qkv, const float* __restrict__ tab,
                                                              bf16* __restrict__ out, BatchView bv, KvView kv, int Hq,
                                                              float scale_log2) {
    constexpr int RW = 4 / SETS;         // waves along the rows
    constexpr int BQ = 32 * RW, BK = 64;
    constexpr int DB = D / 32;           // 32-wide blocks of the head dim
    constexpr int KS = D / 16;           // MFMA k-steps over the head dim
    constexpr int BLK = 32 * D;          // elements per cache block
    constexpr int NL = D / 32 * SETS;    // 1 KiB DMA loads per wave per tile, for K and again for V
    constexpr int STAGE = 4 * BLK;       // elements per stage: K tile (2 blocks) then V tile (2 blocks)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

    // Workgroups go to the eight XCDs in turn.  With a multiple of 8 heads, XCD x takes Hq / 8 consecutive
    // heads; it walks them kv group by kv group, and inside a group query tile by query tile with the group's
    // heads next to each other: the workgroups that run on an XCD at the same time then read the K and V of
    // one kv head (of a few sequences) and find them in that XCD's L2.  (Dealt out head by head across the
    // XCDs, every L2 fetched every K and V: 2.6 times the algorithmic traffic, and 11 % (MHA) to 21 % (8
    // query heads per kv head) more time.)
    int item, h, sub;                                        // sub: which BQ rows of the item's
    if ((Hq & 7) == 0) {
        const int xcd = blockIdx.x & 7;
        int seq = blockIdx.x >> 3;
        sub = seq % SETS;
        seq /= SETS;
        const int hpx = Hq >> 3, G = Hq / kv.Hkv;
        // A grid that fits the chip's slots in one go (two workgroups per CU, 64 per XCD) lasts as long as its
        // busiest CU.  An XCD's CUs take its workgroups 0..31 first and 32.. as their second one, so CU c holds
        // workgroups c and 32 + c; with the items ordered longest first that pairs long with long.  The second
        // half is therefore walked backwards: CU c gets the c-th longest and the c-th shortest (one 2000-token
        // sequence: 73 -> 60 us).  Larger grids are handed out as slots free up; longest first is right there.
        const int n_x = bv.n_prefill_items * hpx;
        if (SETS == 1 && n_x <= 64 && seq >= 32) seq = 32 + (n_x - 1 - seq);
        // heads of one kv group that sit next to each other on this XCD (1 if groups do not tile its heads)
        const int gl = G >= hpx ? hpx : (hpx % G == 0 ? G : 1);
        const int per_group = bv.n_prefill_items * gl;
        const int grp = seq / per_group, r = seq - grp * per_group;
        item = r / gl;
        h = xcd * hpx + grp * gl + (r - item * gl);
    } else {
        sub = blockIdx.x % SETS;
        h = blockIdx.x / (bv.n_prefill_items * SETS);
        item = blockIdx.x / SETS % bv.n_prefill_items;
    }
    const int s = bv.prefill_items[2 * item];
    const int qt = bv.prefill_items[2 * item + 1] * SETS + sub;          // in tiles of BQ rows
    const int q0 = bv.q_start[s];
    const int qlen = bv.q_start[s + 1] - q0;
    if (SETS > 1 && qt * BQ >= qlen) return;
    const int before = bv.kv_before[s];
    const int slot = bv.seq_slot[s];
    const int Hkv = kv.Hkv;
    const int cap = kv.slot_cap[slot];
    const int kvh = h / (Hq / Hkv);
    const size_t head_base = (size_t)kv.slot_off[slot] * Hkv * D + (size_t)kvh * cap * D;
    const bf16* Kc = kv.k + head_base;
    const bf16* Vc = kv.v + head_base;
    const int nqkv = (Hq + 2 * Hkv) * D;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = (tid >> 6) % RW;                        // rows 32 * wave .. of the tile
    const int set = SETS == 1 ? 0 : __builtin_amdgcn_readfirstlane((tid >> 6) / RW);
    bf16* smem = reinterpret_cast<bf16*>(smem_raw) + set * (2 * STAGE);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int lq = lane & 31, lh = lane >> 5;
    const int qi = qt * BQ + wave * 32 + lq;
    const bool valid = qi < qlen;
    const int qic = valid ? qi : qlen - 1;
    const int qpos = before + qic;

    const int last_q = ((qt * BQ + BQ < qlen) ? qt * BQ + BQ : qlen) - 1;
    const int kv_end = before + last_q + 1;                 // keys 0..kv_end-1 are visible to this tile
    const int ntiles = (kv_end + BK - 1) / BK;
    const int last_blk = (kv_end - 1) >> 5;
    int wq_first = qt * BQ + wave * 32, wq_last = wq_first + 31;
    if (wq_last > qlen - 1) wq_last = qlen - 1;
    if (wq_first > qlen - 1) wq_first = qlen - 1;
    const int wave_max_pos = before + wq_last, wave_min_pos = before + wq_first;

    // tile -> LDS: wave w moves 1 KiB pieces w*NL .. w*NL+NL-1 of the K tile and of the V tile.  A
    // block past the last visible one is replaced by the last visible block (its scores are masked).
    // load q in [0, 2*NL) of a tile: K pieces first (needed first), then V pieces
    auto issue_one = [&](int tile, int stage, int q) {
        bf16* st = smem + stage * STAGE;
        const int j = q % NL;
        const int piece = wave_u * NL + j;                   // 512 elements each
        const int blk = piece / (BLK / 512), off = (piece % (BLK / 512)) * 512;
        int kb = tile * 2 + blk;
        if (kb > last_blk) kb = last_blk;
        const size_t src = (size_t)kb * BLK + off + lane * 8;
        if (q < NL) __builtin_amdgcn_global_load_lds((gptr_t)(Kc + src), (lptr_t)(st + piece * 512), 16, 0, 0);
        else __builtin_amdgcn_global_load_lds((gptr_t)(Vc + src), (lptr_t)(st + 2 * BLK + piece * 512), 16, 0, 0);
    };
    auto issue = [&](int tile, int stage) {
#pragma unroll
        for (int q = 0; q < 2 * NL; ++q) issue_one(tile, stage, q);
    };
    issue(set, 0);

    bf16x8 qf[KS];
    load_query<D, ROTATED>(qkv + (size_t)(q0 + qic) * nqkv + h * D, tab + (size_t)qpos * D, qf, lh);

    f32x16 o[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    float m = -INFINITY, l = 0.f;           // running max (already scaled) and sum of this lane's query row

    const int rounds = (ntiles + SETS - 1) / SETS;
    for (int i = 0; i < rounds; ++i) {
        const int tile = i * SETS + set;                     // one past the last for the second set at times: wholly masked
        const int kbase = tile * BK;
        __builtin_amdgcn_s_waitcnt(0x0070);                  // own pieces of this tile landed, own LDS reads done
        __syncthreads();                                     // everyone's pieces landed; the other stage is free
        // after the last tile the same tile is requested once more into the idle stage: the load schedule
        // then needs no branch between the MFMAs
        const int nxt = i + 1 < rounds ? tile + SETS : tile;
        if (kbase > wave_max_pos) {                          // wave-uniform: tile fully masked for this wave
            issue(nxt, (i + 1) & 1);
        } else {
            const bf16* Ks = smem + (i & 1) * STAGE;
            const bf16* Vs = Ks + 2 * BLK;
            f32x16 sacc[2];
            // Operand fetch runs ahead of the MFMAs by hand: written as "read, multiply" the compiler waits for
            // every LDS read right before its MFMA, and the score phase takes 2.6 times its 16 MFMAs.  Here the
            // eight K fragments of the first key block are requested together; each is replaced by the second
            // block's fragment as soon as its MFMA has gone, and under the second block's MFMAs the V fragments
            // of the first two k-steps of P.V are requested.
            // The next tile's loads go out one by one between the score MFMAs: a load holds the wave's
            // instruction stream for tens of cycles, which an MFMA in flight covers.
            constexpr int EVERY = (2 * KS) / (2 * NL);
            auto k_frag = [&](int kb, int ks) {
                return *reinterpret_cast<const bf16x8*>(&Ks[kb * BLK + ((ks * 2 + lh) * 32 + lq) * 8]);
            };
            auto v_frag = [&](int t, int b) {
                return *reinterpret_cast<const bf16x8*>(&Vs[(t >> 1) * BLK + ((2 * (t & 1) + lh) * D + b * 32 + lq) * 8]);
            };
            bf16x8 ka[KS], vfr[2][DB];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) ka[ks] = k_frag(0, ks);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) sacc[kb][r] = 0.f;
            __builtin_amdgcn_sched_barrier(0);             // the order below is the order wanted: nothing is moved across
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qf[ks], sacc[kb], 0, 0, 0);
                    if (kb == 0) ka[ks] = k_frag(1, ks);
                    else if (ks < 2 * DB) vfr[ks / DB][ks % DB] = v_frag(ks / DB, ks % DB);
                    const int m = kb * KS + ks;
                    if (m % EVERY == EVERY - 1) issue_one(nxt, (i + 1) & 1, m / EVERY);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (kbase + BK - 1 > wave_min_pos) {             // wave-uniform: the diagonal crosses this tile
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int kvi = kbase + kb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                        if (kvi > qpos) sacc[kb][r] = -INFINITY;
                    }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[kb][r]);
            mx = fmaxf(m, mx * scale_log2);                  // scale > 0: max commutes with it
            mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
            // a row may have seen no key yet in the second set's tiles
            const float ref = SETS == 1 || mx > -INFINITY ? mx : 0.f;
            if (__builtin_amdgcn_ballot_w64(mx != m) != 0) { // some row's max moved: rescale (wave-uniform)
                const float alpha = fast_exp2(m - ref);      // m = -inf on the first tile -> 0
                l *= alpha;
#pragma unroll
                for (int b = 0; b < DB; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
                m = mx;
            }
            float rs = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float p = fast_exp2(fmaf(sacc[kb][r], scale_log2, -ref));
                    sacc[kb][r] = p;
                    rs += p;
                }
            rs += __shfl_xor(rs, 32, kWave);
            l += rs;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                bf16x8 pf;
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[e] = (bf16)sacc[t >> 1][8 * (t & 1) + e];
#pragma unroll
                for (int b = 0; b < DB; ++b) {
                    o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr[t & 1][b], pf, o[b], 0, 0, 0);
                    if (t + 2 < 4) vfr[t & 1][b] = v_frag(t + 2, b);
                }
            }
        }
    }

    __builtin_amdgcn_s_waitcnt(0x0F70);                      // no LDS write may be in flight when the workgroup ends
    if (SETS == 2) {
        // value r of thread t of a set at ex[TS r + t]
        constexpr int TS = 64 * RW;
        float* ex = reinterpret_cast<float*>(smem_raw) + tid % TS;
        static_assert((DB * 16 + 2) * TS * (int)sizeof(float) <= SETS * 2 * STAGE * (int)sizeof(bf16) || SETS == 1, "merge buffer");
        __syncthreads();                                     // everyone's loads landed and operands are read
        if (set == 1) {
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) ex[(b * 16 + r) * TS] = o[b][r];
            ex[DB * 16 * TS] = m;
            ex[(DB * 16 + 1) * TS] = l;
        }
        __syncthreads();
        if (set == 1) return;
        const float m2 = ex[DB * 16 * TS], l2 = ex[(DB * 16 + 1) * TS];
        const float M = fmaxf(m, m2);                        // finite: the first set has seen key 0
        const float f1 = fast_exp2(m - M), f2 = fast_exp2(m2 - M);
        l = l * f1 + l2 * f2;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[b][r] = o[b][r] * f1 + ex[(b * 16 + r) * TS] * f2;
    }
    if (valid) {
        const float inv = 1.0f / l;
        bf16* op = out + (size_t)(q0 + qi) * Hq * D + h * D;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                bf16x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = (bf16)(o[b][r4 * 4 + e] * inv);
                *reinterpret_cast<bf16x4*>(op + b * 32 + 8 * r4 + 4 * lh) = w;
            }
    }
}

template <int D, bool ROTATED, int SETS>
static void launch_prefill_sets(const act_t* qkv, const float* rope_tab, act_t* out, const BatchView& bv, const KvView& kv,
                                int Hq, hipStream_t st) {
    constexpr int kLds = SETS * 2 * 4 * 32 * D * (int)sizeof(bf16);     // per set two stages of (K tile + V tile)
    static LdsLimit limit;
    if (!limit.raise(reinterpret_cast<const void*>(attn_prefill_kernel<D, ROTATED, SETS>), kLds) && SETS > 1)
        return launch_prefill_sets<D, ROTATED, 1>(qkv, rope_tab, out, bv, kv, Hq, st);
    const float scale_log2 = kLog2e / sqrtf((float)D);
    hipLaunchKernelGGL((attn_prefill_kernel<D, ROTATED, SETS>), dim3(bv.n_prefill_items * Hq * SETS), dim3(256), kLds, st, qkv,
                       rope_tab, out, bv, kv, Hq, scale_log2);
}

// 64-row workgroups with two sets of waves while a CU gets one of them at most and the chains are long enough to pay for
// the merge: from four KV tiles on.  Their time over that of 128-row tiles (seven head counts of both sizes, 20 to 512 rows in one
// or two sequences): 1.21 at one KV tile, 1.02 at two and three (0.93 to 1.14), 0.91 at four (0.84 to 1.02), 0.93 at five, 0.81 at
// eight, 0.72 at 16, 0.63 at 56.  (The second set as four more waves on the same CU: 78 -> 71 us instead of 56 at 55 tiles, and
// 12.2 -> 16.9 at 3 to 5.)
constexpr int kLongKeys = 192;
template <int D, bool ROTATED>
static void launch_prefill_d(const act_t* qkv, const float* rope_tab, act_t* out, const BatchView& bv, const KvView& kv,
                             int Hq, hipStream_t st) {
    if (bv.n_prefill_items * Hq <= 128 && bv.prefill_keys > kLongKeys)
        launch_prefill_sets<D, ROTATED, 2>(qkv, rope_tab, out, bv, kv, Hq, st);
    else launch_prefill_sets<D, ROTATED, 1>(qkv, rope_tab, out, bv, kv, Hq, st);
}

void launch_attn_prefill(const QkvSource& src, const float* rope_tab, act_t* out, const BatchView& bv, const KvView& kv,
                         int Hq, hipStream_t st) {
    if (bv.n_prefill_items <= 0) return;
    const bool rotated = src.partial != nullptr;
    if (kv.d == 128) (rotated ? launch_prefill_d<128, true> : launch_prefill_d<128, false>)(src.qkv, rope_tab, out, bv, kv, Hq, st);
    else (rotated ? launch_prefill_d<64, true> : launch_prefill_d<64, false>)(src.qkv, rope_tab, out, bv, kv, Hq, st);
}

#else  // BZ_FP32_DEBUG
// ---------------------------------------------------------------------------------------------
// fp32 debug prefill: one wave per (token, head); scores for all visible keys are kept in LDS and
// softmax is the plain three-pass form.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void attn_naive_kernel(const float* __restrict__ qkv, float* __restrict__ out,
                                                        BatchView bv, KvView kv, int Hq, float scale_log2) {
    extern __shared__ float sc[];
    const int t = blockIdx.x, h = blockIdx.y;
    const int s = bv.token_seq[t];
    if (bv.q_start[s + 1] - bv.q_start[s] <= 1) return;     // single-token sequences use the decode kernel
    const int pos = bv.kv_before[s] + (t - bv.q_start[s]);
    const int slot = bv.seq_slot[s];
    const int D = kv.d, Hkv = kv.Hkv, cap = kv.slot_cap[slot];
    const int kvh = h / (Hq / Hkv);
    const size_t head_base = (size_t)kv.slot_off[slot] * Hkv * D + (size_t)kvh * cap * D;
    const float* Kc = kv.k + head_base;
    const float* Vc = kv.v + head_base;
    const float* q = qkv + (size_t)t * (Hq + 2 * Hkv) * D + h * D;
    const int lane = threadIdx.x;
    float mx = -INFINITY;
    for (int j = lane; j <= pos; j += 64) {
        float a = 0.f;
        for (int e = 0; e < D; ++e) a = fmaf(q[e], Kc[k_elem_offset(j, e, D)], a);
        a *= scale_log2;
        sc[j] = a;
        mx = fmaxf(mx, a);
    }
    mx = wave_max(mx);
    float sum = 0.f;
    for (int j = lane; j <= pos; j += 64) {
        const float p = exp2f(sc[j] - mx);
        sc[j] = p;
        sum += p;
    }
    sum = wave_sum(sum);
    __syncthreads();
    for (int e = lane; e < D; e += 64) {
        float a = 0.f;
        for (int j = 0; j <= pos; ++j) a = fmaf(sc[j], Vc[v_elem_offset(j, e, D)], a);
        out[(size_t)t * Hq * D + h * D + e] = a / sum;
    }
}

void launch_attn_prefill(const QkvSource& qkv, const float*, act_t* out, const BatchView& bv, const KvView& kv, int Hq,
                         hipStream_t st) {
    if (bv.n_prefill_items <= 0) return;
    const float scale_log2 = kLog2e / sqrtf((float)kv.d);
    // 64 KiB of LDS holds 16384 scores: enough for every supported max_seq_len in the debug build
    static LdsLimit limit;
    (void)limit.raise(reinterpret_cast<const void*>(attn_naive_kernel), 65536);
    hipLaunchKernelGGL(attn_naive_kernel, dim3(bv.T, Hq), dim3(64), 65536, st, qkv.qkv, out, bv, kv, Hq, scale_log2);
}
#endif

// ---------------------------------------------------------------------------------------------
// Decode.  Grid (chunk, kv head, decode sequence).  A workgroup handles kDecodeChunk = 256 cached
// positions of one kv head for all G = Hq/Hkv query heads that share it: every K and V byte is
// read from HBM once.  Each of the 4 waves owns 64 positions and runs on its own until the four
// partial results are merged.  Each workgroup writes an unnormalised partial (o, running max, sum)
// per head; the combine kernel folds the chunks of a sequence in increasing chunk order, so the
// result does not depend on scheduling.
// ---------------------------------------------------------------------------------------------
#ifndef BZ_FP32_DEBUG
constexpr int kDecodeMaxG = 8;

// Both products run on the matrix cores with the cache as the row operand, read from global
// memory straight into the instructions (a lane's 16 bytes are one operand register pair):
//   S^T[pos, g] = K[pos, :] . q[g, :]     q fills G of the 32 columns, the rest are zero;
//   O^T[j, g]   = V^T[j, pos] . P^T[pos, g]   P^T goes from the score accumulators to the column
//   operand inside the registers (the V cache is stored in the matching position order).
//
// The new token's rotation and its append to the cache happen here too, in the shadow of the stream: the projection's
// values are requested before the workgroup's K and V, four pairs per thread, and go through LDS to the waves.  The
// workgroup whose chunk holds the new position rotates and appends K and V and adds the position as a fifth partial
// result (score from a plain dot product, probability 1 against its own maximum); everywhere else only cached positions
// count.  A launch of its own for these few bytes per sequence cost 5 to 7.5 us of a 105 to 370 us decode layer.
// A sequence with a single chunk gets its output here; the combine kernel leaves it alone.
//
// SRC: what the new token's values come as: the projection, its partial sums, or rotated and appended already
// (decode_append_apart).  In the last case the queries come in one of two ways.  On caches of up to four chunks on average (kAppended)
// they are requested before the stream, by the first 128 threads, and go through LDS; the store waits for the wave's whole stream (not
// all waves request one), so the scores start when K and V are there.  On longer ones (kAppendedLong) every wave requests them for
// itself, behind its stream.  A pass of two layers, behind the stream against through LDS, same memory: 7B shape, 161 sequences of
// 128 to 1024 positions 919 / 902 us, of 511 806 / 802, of 900 to 1023 1193 / 1187, of 1023 1240 / 1245, 150 of 1500 to 3000 2094 / 2104; 13B
// shape, 83 of 512 to 4096 1561 / 1575, of 2047 1423 / 1440.  Products that start as K arrives are slower than either where
// chunks are full: stored behind a counted wait 1272 (of 1023), 2108, 1590, 1477; by every wave into LDS of its own 1250, 2110, 1571, 1449.
// WAVES per SIMD, that is workgroups per CU, set outright: for d = 128 two keep the memory streams in longer runs than three,
// which the registers would allow where the projection is plain (83 sequences of 40 heads, 402 -> 392 us; 240 of 8 with four
// query heads each 371 -> 366), except where most caches end within their first chunk (250 sequences of 40 heads 178 -> 170 with
// three).
enum { kProjection = 0, kPartialSums = 1, kAppended = 2, kAppendedLong = 3 };
template <int D, int SRC, int WAVES>
__global__ __attribute__((amdgpu_waves_per_eu(WAVES, WAVES))) __launch_bounds__(256) void attn_decode_kernel(QkvSource src, const float* __restrict__ tab,
                                                             float* __restrict__ partial, bf16* __restrict__ out,
                                                             BatchView bv, KvView kv, int Hq, int G, float scale_log2,
                                                             int combine) {
    constexpr int CH = kDecodeChunk;
    constexpr int KS = D / 16, DB = D / 32, BLK = 32 * D;
    constexpr bool REDUCE = SRC == kPartialSums, FUSED = SRC < kAppended, HANDED = SRC != kAppendedLong;
    __shared__ float wmx[4][kDecodeMaxG];
    __shared__ float wsum[4][kDecodeMaxG];
    __shared__ float osh[4][kDecodeMaxG][D];
    __shared__ __attribute__((aligned(16))) bf16 qs[kDecodeMaxG][D];       // rotated queries
    __shared__ __attribute__((aligned(16))) bf16 kn[D], vn[D];             // the new position's key and value
    __shared__ float sn[kDecodeMaxG];                                      // its scores

    // the work list names only chunks that exist, and brings the sequence's slot along: everything else
    // hangs off one more level of loads (see BatchView for the order of workgroups)
    const int e = blockIdx.x / kv.Hkv;
    const int4 item = bv.decode_work[2 * e], item2 = bv.decode_work[2 * e + 1];
    const int s = item.x, slot = item.y, di = item.z;
    const int rest = blockIdx.x - kv.Hkv * item2.x;          // position among this sequence's (kv head, chunk) pairs
    const int kvh = rest / item.w, chunk = rest - kvh * item.w;
    const int pos = bv.kv_before[s];                         // the new token's position
    const int cached = FUSED ? pos : pos + 1;
    const int c0 = chunk * CH;
    if (c0 > pos) return;
    const bool newest = FUSED && pos - c0 < CH;              // this chunk holds the new position, which is not cached yet
    const int t = bv.q_start[s];
    const int Hkv = kv.Hkv, cap = kv.slot_cap[slot];
    const size_t head_base = (size_t)kv.slot_off[slot] * Hkv * D + (size_t)kvh * cap * D;
    bf16* Kc = kv.k + head_base;
    bf16* Vc = kv.v + head_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, lh = lane >> 5;

    // unit = 4 pairs (j, j + D/2) of one of the G query heads or (newest) of the key, or 4 values (newest); threads past
    // the last unit repeat it and store nothing but the same LDS values
    constexpr int UPH = D / 8;
    const int n_rot = (newest ? G + 1 : G) * UPH, n_units = newest ? n_rot + D / 4 : n_rot;
    const int unit = tid < n_units ? tid : n_units - 1;
    const bool is_v = unit >= n_rot;
    const int hh = is_v ? 0 : unit / UPH;
    const int j0 = (is_v ? unit - n_rot : unit - hh * UPH) * 4;
    const int nqkv = (Hq + 2 * Hkv) * D;
    const size_t slice = (size_t)bv.T * nqkv;
    const size_t at = (size_t)t * nqkv + (is_v ? Hq + Hkv + kvh : hh < G ? kvh * G + hh : Hq + kvh) * D + j0;
    const int second = is_v ? 0 : D / 2;
    const float* cs = tab + (size_t)pos * D + (is_v ? 0 : j0 * 2);
    f32x4 pa[4], pb[4], cs0, cs1;                            // REDUCE: up to four slices, the rest later
    bf16x4 ra, rb;
    if (REDUCE) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float* p = src.partial + (k < src.ksplit ? k : src.ksplit - 1) * slice + at;
            pa[k] = *reinterpret_cast<const f32x4*>(p);
            pb[k] = *reinterpret_cast<const f32x4*>(p + second);
        }
    } else if (FUSED) {
        ra = *reinterpret_cast<const bf16x4*>(src.qkv + at);
        rb = *reinterpret_cast<const bf16x4*>(src.qkv + at + second);
    }
    bf16x8 qr;                                               // kAppended: 8 values of the G * D, at most 128 threads' worth
    if (FUSED) {
        cs0 = *reinterpret_cast<const f32x4*>(cs);
        cs1 = *reinterpret_cast<const f32x4*>(cs + 4);
    } else if (HANDED) {
        const int i = tid < G * (D / 8) ? tid : G * (D / 8) - 1;
        qr = *reinterpret_cast<const bf16x8*>(src.qkv + (size_t)t * nqkv + kvh * G * D + i * 8);
    }
    __builtin_amdgcn_sched_barrier(0);                       // these go out before the stream

    const int w0 = c0 + wave * 64;
    const bool live = w0 < cached;                           // something cached in this wave's range; wave-uniform
    // The loads stand outside any branch, or the wait for the projection's values would have to assume that they were not
    // issued and drain them.  A block past the end is replaced by the last valid one (its positions get probability zero);
    // a wave without cached positions reads one line per load, of block 0, or (nothing to wait for before) nothing.
    const int last_blk = live ? (cached - 1) >> 5 : 0;
    const int lane_k = live ? (lh * 32 + lq) * 8 : 0, lane_v = live ? (lh * D + lq) * 8 : 0;
    size_t boff[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        int kb = (w0 >> 5) + b;
        if (kb > last_blk) kb = last_blk;
        boff[b] = (size_t)kb * BLK;
    }
    bf16x8 kf[2][KS], vf[2][2][DB];
    if (FUSED || live) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                kf[b][ks] = stream_load(reinterpret_cast<const bf16x8*>(Kc + boff[b] + lane_k + ks * 512));
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    vf[b][tt][db] =
                        stream_load(reinterpret_cast<const bf16x8*>(Vc + boff[b] + lane_v + (2 * tt * D + db * 32) * 8));
    }
    bf16x8 qa[KS];
    if (!HANDED && live) {
        const bf16* q = src.qkv + (size_t)t * nqkv + kvh * G * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (lq < G) qa[ks] = *reinterpret_cast<const bf16x8*>(q + lq * D + ks * 16 + lh * 8);
            else
#pragma unroll
                for (int i = 0; i < 8; ++i) qa[ks][i] = (bf16)0.f;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (FUSED) {
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
        if (REDUCE) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < src.ksplit) {
                    a += pa[k];
                    b += pb[k];
                }
            for (int k = 4; k < src.ksplit; ++k) {
                a += *reinterpret_cast<const f32x4*>(src.partial + k * slice + at);
                b += *reinterpret_cast<const f32x4*>(src.partial + k * slice + at + second);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = (float)(bf16)a[i];
                b[i] = (float)(bf16)b[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = (float)ra[i];
                b[i] = (float)rb[i];
            }
        }
        if (is_v) {
            bf16x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (bf16)a[i];
            *reinterpret_cast<bf16x4*>(&vn[j0]) = v;
            if (tid < n_units) {
#pragma unroll
                for (int i = 0; i < 4; ++i) Vc[v_elem_offset(pos, j0 + i, D)] = v[i];
            }
        } else {
            bf16x4 lo, hi;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float c = i < 2 ? cs0[2 * i] : cs1[2 * i - 4], sv = i < 2 ? cs0[2 * i + 1] : cs1[2 * i - 3];
                lo[i] = (bf16)(a[i] * c - b[i] * sv);
                hi[i] = (bf16)(b[i] * c + a[i] * sv);
            }
            bf16* dst = hh < G ? qs[hh] : kn;
            *reinterpret_cast<bf16x4*>(dst + j0) = lo;
            *reinterpret_cast<bf16x4*>(dst + D / 2 + j0) = hi;
            if (hh == G && tid < n_units) {
                *reinterpret_cast<bf16x4*>(Kc + k_elem_offset(pos, j0, D)) = lo;
                *reinterpret_cast<bf16x4*>(Kc + k_elem_offset(pos, D / 2 + j0, D)) = hi;
            }
        }
    }
    if (!FUSED && HANDED && tid < G * (D / 8)) *reinterpret_cast<bf16x8*>(&qs[0][0] + tid * 8) = qr;
    if (HANDED) {
        // hand-over through LDS; a full barrier would drain the stream
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
    if (newest) {                                            // workgroup-uniform
        for (int g = wave; g < G; g += 4) {
            float p = 0.f;
#pragma unroll
            for (int i = 0; i < D / kWave; ++i) p = fmaf((float)qs[g][lane * (D / kWave) + i], (float)kn[lane * (D / kWave) + i], p);
            p = wave_sum(p);
            if (lane == 0) sn[g] = p * scale_log2;
        }
    }
    if (live) {
        f32x16 sacc[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) sacc[b][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 qf = {};
            if (!HANDED) qf = qa[ks];
            else if (lq < G) qf = *reinterpret_cast<const bf16x8*>(&qs[lq][ks * 16 + lh * 8]);
#pragma unroll
            for (int b = 0; b < 2; ++b) sacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[b][ks], qf, sacc[b], 0, 0, 0);
        }
        // lane (g = lane%32, h = lane/32) holds positions b*32 + 8*(r/4) + 4h + r%4 of head g
        float m = -INFINITY;
        if (w0 + 64 > cached) {                              // wave-uniform: the range ends here
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (w0 + b * 32 + 8 * (r >> 2) + 4 * lh + (r & 3) >= cached) sacc[b][r] = -INFINITY;
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) m = fmaxf(m, sacc[b][r]);
        m = fmaxf(m, __shfl_xor(m, 32, kWave)) * scale_log2; // finite: position w0 is valid; scale > 0
        float l = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                // not the bare hardware exponential: weights below the normal range count too (0.1 to 0.3 us of 7.2 to 272)
                const float p = exp2f(fmaf(sacc[b][r], scale_log2, -m));
                sacc[b][r] = p;
                l += p;
            }
        l += __shfl_xor(l, 32, kWave);
        f32x16 oacc[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                bf16x8 pf;
#pragma unroll
                for (int i = 0; i < 8; ++i) pf[i] = (bf16)sacc[b][8 * tt + i];
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[b][tt][db], pf, oacc[db], 0, 0, 0);
            }
        if (lq < G) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                    *reinterpret_cast<float4*>(&osh[wave][lq][db * 32 + 8 * r4 + 4 * lh]) =
                        make_float4(oacc[db][4 * r4], oacc[db][4 * r4 + 1], oacc[db][4 * r4 + 2], oacc[db][4 * r4 + 3]);
            if (lh == 0) {
                wmx[wave][lq] = m;
                wsum[wave][lq] = l;
            }
        }
    } else {
        for (int i = lane; i < G * D; i += 64) osh[wave][i / D][i % D] = 0.f;
        if (lane < G) {
            wmx[wave][lane] = -INFINITY;
            wsum[wave][lane] = 0.f;
        }
    }
    __syncthreads();
    // merge the four waves in wave order, then the new position
    const int PS = decode_partial_stride(D);
    const bool alone = item.w == 1 && combine;               // the sequence's only chunk: the output itself
    for (int i = tid; i < G * D; i += 256) {
        const int g = i / D, dd = i - g * D;
        float M = fmaxf(fmaxf(wmx[0][g], wmx[1][g]), fmaxf(wmx[2][g], wmx[3][g]));
        if (newest) M = fmaxf(M, sn[g]);
        float acc = 0.f, L = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float f = exp2f(wmx[w][g] - M);
            acc = fmaf(osh[w][g][dd], f, acc);
            L = fmaf(wsum[w][g], f, L);
        }
        if (newest) {
            const float f = exp2f(sn[g] - M);
            acc = fmaf((float)vn[dd], f, acc);
            L += f;
        }
        if (alone) {
            out[(size_t)t * Hq * D + (kvh * G + g) * D + dd] = (bf16)(acc / L);
        } else {
            float* pp = partial + (((size_t)di * Hq + kvh * G + g) * bv.decode_chunks + chunk) * PS;
            pp[dd] = acc;
            if (dd == 0) {
                pp[D] = M;
                pp[D + 1] = L;
            }
        }
    }
}

#else
// fp32 debug build: scores with one lane per position, PV with D/8 lanes per position, on the VALU.
template <int D, int G>
__global__ __launch_bounds__(256) void attn_decode_kernel(const float* __restrict__ qkv, float* __restrict__ partial,
                                                          BatchView bv, KvView kv, int Hq, int, float scale_log2) {
    constexpr int CH = kDecodeChunk;
    constexpr int LPR = D / 8;            // lanes per position in the PV product
    constexpr int RPI = 64 / LPR;         // positions per wave step
    constexpr int NSTEP = 64 / RPI;       // steps for the wave's 64 positions
    __shared__ float ps[4][G][64];
    __shared__ float wmx[4][G];
    __shared__ float wsum[4][G];
    __shared__ float osh[4][G][D];
    __shared__ float qs[G][D];

    // the work list names only chunks that exist, and brings the sequence's slot along: everything else
    // hangs off one more level of loads (see BatchView for the order of workgroups)
    const int e = blockIdx.x / kv.Hkv;
    const int4 item = bv.decode_work[2 * e], item2 = bv.decode_work[2 * e + 1];
    const int s = item.x, slot = item.y, di = item.z;
    const int rest = blockIdx.x - kv.Hkv * item2.x;          // position among this sequence's (kv head, chunk) pairs
    const int kvh = rest / item.w, chunk = rest - kvh * item.w;
    const int len = bv.kv_before[s] + 1;
    const int c0 = chunk * CH;
    if (c0 >= len) return;
    const int t = bv.q_start[s];
    const int Hkv = kv.Hkv, cap = kv.slot_cap[slot];
    const size_t head_base = (size_t)kv.slot_off[slot] * Hkv * D + (size_t)kvh * cap * D;
    const float* Kc = kv.k + head_base;
    const float* Vc = kv.v + head_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* q = qkv + (size_t)t * (Hq + 2 * Hkv) * D + (size_t)kvh * G * D;
    const int w0 = c0 + wave * 64;
    const int sub = lane / LPR, dv = (lane % LPR) * 8;
    {
        for (int i = tid; i < G * D / 8; i += 256) {
            float v[8];
            load8(q + i * 8, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) (&qs[0][0])[i * 8 + e] = v[e];
        }
        __syncthreads();
        const int pos = w0 + lane;
        const bool valid = pos < len;
        const int kpos = valid ? pos : len - 1;
        float sc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) sc[g] = 0.f;
        for (int c = 0; c < D / 8; ++c) {
            float kk[8];
            load8(Kc + k_piece_offset(kpos, c, D), kk);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 8; ++e) sc[g] = fmaf(kk[e], qs[g][c * 8 + e], sc[g]);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float sg = valid ? sc[g] * scale_log2 : -INFINITY;
            const float m = wave_max(sg);
            const float p = valid ? exp2f(sg - m) : 0.f;
            ps[wave][g][lane] = p;
            const float l = wave_sum(p);
            if (lane == 0) {
                wmx[wave][g] = m;
                wsum[wave][g] = l;
            }
        }
    }

    float o[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e) o[g][e] = 0.f;
    for (int stp = 0; stp < NSTEP; ++stp) {
        const int prow = stp * RPI + sub;
        int vp = w0 + prow;
        if (vp > len - 1) vp = len - 1;                  // probability zero there
        float vf[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) vf[e] = Vc[v_elem_offset(vp, dv + e, D)];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float pw = ps[wave][g][prow];           // written by this wave only
#pragma unroll
            for (int e = 0; e < 8; ++e) o[g][e] = fmaf(pw, vf[e], o[g][e]);
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = o[g][e];
#pragma unroll
            for (int off = LPR; off < 64; off <<= 1) v += __shfl_xor(v, off, kWave);
            o[g][e] = v;
        }
    if (lane < LPR) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) osh[wave][g][dv + e] = o[g][e];
    }
    __syncthreads();
    // merge the four waves in wave order
    const int PS = decode_partial_stride(D);
    for (int i = tid; i < G * D; i += 256) {
        const int g = i / D, dd = i - g * D;
        const float M = fmaxf(fmaxf(wmx[0][g], wmx[1][g]), fmaxf(wmx[2][g], wmx[3][g]));
        float acc = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) acc = fmaf(osh[w][g][dd], exp2f(wmx[w][g] - M), acc);
        partial[(((size_t)di * Hq + kvh * G + g) * bv.decode_chunks + chunk) * PS + dd] = acc;
    }
    if (tid < G) {
        const int g = tid;
        const float M = fmaxf(fmaxf(wmx[0][g], wmx[1][g]), fmaxf(wmx[2][g], wmx[3][g]));
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) L = fmaf(wsum[w][g], exp2f(wmx[w][g] - M), L);
        float* pp = partial + (((size_t)di * Hq + kvh * G + g) * bv.decode_chunks + chunk) * PS;
        pp[D] = M;
        pp[D + 1] = L;
    }
}

#endif

// One workgroup per (decode sequence, head), one thread per head-dim index.  Chunks are folded in
// increasing order, sixteen per batch: all loads of a batch are independent (an index past the end
// re-reads the last chunk; its value is not added), so a sequence of up to 4096 positions costs one
// memory round trip.  Across batches the running (max, numerator, denominator) is rescaled.
template <int D>
__global__ __launch_bounds__(D) void attn_combine_kernel(const float* __restrict__ partial, act_t* __restrict__ out,
                                                         BatchView bv, int Hq) {
    constexpr int NB = 16;
    const int di = blockIdx.x, h = blockIdx.y, dd = threadIdx.x;
    const int s = bv.decode_seqs[di];
    const int len = bv.kv_before[s] + 1;
    const int nch = (len + kDecodeChunk - 1) / kDecodeChunk;
#ifndef BZ_FP32_DEBUG
    if (nch == 1) return;                                    // the decode kernel has written the output
#endif
    const int PS = decode_partial_stride(D);
    const float* base = partial + ((size_t)di * Hq + h) * bv.decode_chunks * PS;
    float M = -INFINITY, num = 0.f, den = 0.f;
    for (int c0 = 0; c0 < nch; c0 += NB) {
        float mv[NB], ov[NB], lv[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const float* pc = base + ((c0 + u < nch) ? c0 + u : nch - 1) * PS;
            mv[u] = pc[D];
            ov[u] = pc[dd];
            lv[u] = pc[D + 1];
        }
        float Mb = M;
#pragma unroll
        for (int u = 0; u < NB; ++u) Mb = fmaxf(Mb, mv[u]);
        const float keep = exp2f(M - Mb);                // 0 for the first batch (M = -inf)
        num *= keep;
        den *= keep;
        M = Mb;
        // no branches here: behind one the compiler moves each load next to its use and the batch turns
        // into sixteen round trips.  A chunk past the end gets weight zero and adds exactly nothing.
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const float w = (c0 + u < nch) ? exp2f(mv[u] - M) : 0.f;
            num = fmaf(ov[u], w, num);
            den = fmaf(lv[u], w, den);
        }
    }
    act_t r;
    from_f32(r, num / den);
    out[(size_t)bv.q_start[s] * Hq * D + h * D + dd] = r;
}

template <int D>
static void launch_decode_d(const QkvSource& qkv, [[maybe_unused]] const float* rope_tab, act_t* out, float* partial,
                            const BatchView& bv, const KvView& kv, int Hq, bool combine, hipStream_t st) {
    const float scale_log2 = kLog2e / sqrtf((float)D);
    const dim3 grid(bv.n_decode_work * kv.Hkv);
    const int G = Hq / kv.Hkv;                      // 1, 2, 4 or 8: checked when the instance is created
#ifndef BZ_FP32_DEBUG
    constexpr int MANY = D == 128 ? 3 : 4;          // what the registers allow
    constexpr int FEW = D == 128 ? 2 : 4;
    const bool apart = decode_append_apart(bv, kv, Hq);
    auto kern = apart && bv.n_decode_work > 4 * bv.n_decode ? attn_decode_kernel<D, kAppendedLong, FEW>
                : apart                             ? attn_decode_kernel<D, kAppended, FEW>
                : qkv.partial                       ? attn_decode_kernel<D, kPartialSums, FEW>
                : bv.n_decode_work < 2 * bv.n_decode ? attn_decode_kernel<D, kProjection, MANY>
                                                    : attn_decode_kernel<D, kProjection, FEW>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, qkv, rope_tab, partial, out, bv, kv, Hq, G, scale_log2, (int)combine);
    if (bv.n_decode_work == bv.n_decode) return;    // one chunk each: nothing to combine
#else
    const act_t* q = qkv.qkv;
    switch (G) {
        case 1: hipLaunchKernelGGL((attn_decode_kernel<D, 1>), grid, dim3(256), 0, st, q, partial, bv, kv, Hq, G, scale_log2); break;
        case 2: hipLaunchKernelGGL((attn_decode_kernel<D, 2>), grid, dim3(256), 0, st, q, partial, bv, kv, Hq, G, scale_log2); break;
        case 4: hipLaunchKernelGGL((attn_decode_kernel<D, 4>), grid, dim3(256), 0, st, q, partial, bv, kv, Hq, G, scale_log2); break;
        default: hipLaunchKernelGGL((attn_decode_kernel<D, 8>), grid, dim3(256), 0, st, q, partial, bv, kv, Hq, G, scale_log2); break;
    }
#endif
    if (combine) hipLaunchKernelGGL(attn_combine_kernel<D>, dim3(bv.n_decode, Hq), dim3(D), 0, st, partial, out, bv, Hq);
}

void launch_attn_decode(const QkvSource& qkv, const float* rope_tab, act_t* out, float* partial, const BatchView& bv,
                        const KvView& kv, int Hq, bool combine, hipStream_t st) {
    if (bv.n_decode <= 0) return;
    if (kv.d == 128) launch_decode_d<128>(qkv, rope_tab, out, partial, bv, kv, Hq, combine, st);
    else launch_decode_d<64>(qkv, rope_tab, out, partial, bv, kv, Hq, combine, st);
}

}  // namespace bz
