// HBM-bound steps of a decoder layer: RMSNorm, KV-cache append (keys rotated on the way), KV scatter /
// gather for cache import/export, and the decode-batch position bump.
#include "common.h"

namespace bz {

// ---------------------------------------------------------------------------------------------
// RMSNorm: one workgroup per token row.  Sum of squares in fp32 (wave shuffle reduction, then a
// fixed-order sum over the waves), y = (x * rstd) * gain rounded once to the activation type.
// ---------------------------------------------------------------------------------------------
// REDUCE: the row of x is first completed as x + (sum of split-K slices), rounded and stored; the
// norm then works on the rounded values, so its result is bit-identical to a separate norm kernel.
// The first kKeep vectors of a thread (rows up to 8 * kKeep * THREADS elements: every supported
// shape) stay in registers between the two passes together with their gains, so the row makes one
// trip from memory.
template <int THREADS, bool REDUCE>
__global__ __launch_bounds__(THREADS) void rmsnorm_kernel(act_t* __restrict__ x, const float* __restrict__ partial,
                                                          int ksplit, int T, const bf16* __restrict__ gain,
                                                          act_t* __restrict__ y, int H, float eps) {
    constexpr int NW = THREADS / kWave;
    constexpr int kKeep = 4;
    __shared__ float red[NW];
    const int row = blockIdx.x;
    act_t* xr = x + (size_t)row * H;
    act_t* yr = y + (size_t)row * H;
    const int nvec = H >> 3;
    float keep[kKeep][8];
    raw8_bf16 gk[kKeep];
    if (gain != nullptr) {
#pragma unroll
        for (int c = 0; c < kKeep; ++c) {
            const int i = threadIdx.x + c * THREADS;
            if (i < nvec) load_raw8(gain + i * 8, gk[c]);
        }
    }
    float ss = 0.f;
    auto first_pass = [&](int i, float (&v)[8]) {
        load8(xr + i * 8, v);
        if (REDUCE) {
            float s[8];
            reduce8(partial, ksplit, (size_t)T * H, (size_t)row * H + i * 8, s);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = s[e] + v[e];
            store8(xr + i * 8, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) {              // continue with the values as stored
                act_t r;
                from_f32(r, v[e]);
                v[e] = to_f32(r);
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf(v[e], v[e], ss);
    };
#pragma unroll
    for (int c = 0; c < kKeep; ++c) {
        const int i = threadIdx.x + c * THREADS;
        if (i < nvec) first_pass(i, keep[c]);
    }
    for (int i = threadIdx.x + kKeep * THREADS; i < nvec; i += THREADS) {
        float v[8];
        first_pass(i, v);
    }
    if (gain == nullptr) return;
    ss = wave_sum(ss);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) tot += red[w];
    const float rstd = 1.0f / sqrtf(tot / (float)H + eps);
#pragma unroll
    for (int c = 0; c < kKeep; ++c) {
        const int i = threadIdx.x + c * THREADS;
        if (i < nvec) {
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (keep[c][e] * rstd) * raw_get(gk[c], e);
            store8(yr + i * 8, o);
        }
    }
    for (int i = threadIdx.x + kKeep * THREADS; i < nvec; i += THREADS) {
        float v[8], g[8];
        load8(xr + i * 8, v);
        load8(gain + i * 8, g);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (v[e] * rstd) * g[e];
        store8(yr + i * 8, v);
    }
}

void launch_rmsnorm(const act_t* x, const bf16* gain, act_t* y, int T, int H, float eps, hipStream_t st) {
    if (T <= 0) return;
    act_t* xm = const_cast<act_t*>(x);       // not written without REDUCE
    if (H >= 4096 && T <= 256) {             // few rows: more threads per row shorten each thread's chain of loads
        hipLaunchKernelGGL((rmsnorm_kernel<512, false>), dim3(T), dim3(512), 0, st, xm, nullptr, 0, T, gain, y, H, eps);
    } else if (H >= 2048) {
        hipLaunchKernelGGL((rmsnorm_kernel<256, false>), dim3(T), dim3(256), 0, st, xm, nullptr, 0, T, gain, y, H, eps);
    } else {
        hipLaunchKernelGGL((rmsnorm_kernel<64, false>), dim3(T), dim3(64), 0, st, xm, nullptr, 0, T, gain, y, H, eps);
    }
}

void launch_reduce_residual_rmsnorm(act_t* x, const float* partial, int ksplit, const bf16* gain, act_t* y, int T,
                                    int H, float eps, hipStream_t st) {
    if (T <= 0) return;
    if (H >= 4096 && T <= 256) {
        hipLaunchKernelGGL((rmsnorm_kernel<512, true>), dim3(T), dim3(512), 0, st, x, partial, ksplit, T, gain, y, H, eps);
    } else if (H >= 2048) {
        hipLaunchKernelGGL((rmsnorm_kernel<256, true>), dim3(T), dim3(256), 0, st, x, partial, ksplit, T, gain, y, H, eps);
    } else {
        hipLaunchKernelGGL((rmsnorm_kernel<64, true>), dim3(T), dim3(64), 0, st, x, partial, ksplit, T, gain, y, H, eps);
    }
}

// ---------------------------------------------------------------------------------------------
// KV append for the sequences with several new tokens: K is rotated and written to the cache, V is copied to it.
// (Single new tokens are appended by the decode attention kernel, or here row by row: decode_append_apart.)
//
// HBM-bound: the K and V parts of the projection in, the cache out.  A workgroup owns one aligned block of 32 positions
// (the unit in which the cache is contiguous) of one sequence for `heads_per_wg` kv heads, so a head's block is written as
// whole cache lines: K as 16-byte pieces, eight consecutive positions of a piece from the eight rows of a wave's load; V
// as two pieces of 8 positions per thread, gathered from 8 rows.  The rotation's cosines and sines are loaded once per
// workgroup.  Before, one workgroup per token rotated queries too and wrote K in 16-byte pieces; that pass against this one
// (the queries' share went to the prefill kernel): 13B shape, 14 091 rows 226 -> 109 us (5.3 TB/s) and 30 more there, 70B, 8192
// rows 62 -> 18 and 32, 7B, 4973 rows 64 -> 42 and 11.
//
// Partial sums (few rows): the loads of several slices and rows go out together, and queries are folded and rotated here by
// workgroups of their own, coalesced.  Folded row by row with one slice's load behind the other, and the queries by every
// lane of the prefill kernel, the append and the attention took, one kernel after the other, 34.8 us (17 rows, 16 + 2 heads
// of 128, six slices), 26.4 (129 rows, 16 + 4 of 64) and 31.7 (2 x 20 rows on 500 positions, 70B); now 12.5, 13.2 and 20.5.
//
// Item i of the prefill list (sequence, tile of 128 new rows) covers the blocks first + 4 * tile + 0..3 of its sequence;
// an unaligned start can make the sequence touch one block more, which the last item's fifth workgroup takes.
// ---------------------------------------------------------------------------------------------
#ifndef BZ_FP32_DEBUG
constexpr int kAppendBlocks = 5;

__device__ __forceinline__ void load_cos_sin(const float* cs, float (&c8)[8], float (&s8)[8]) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const float4 v = *reinterpret_cast<const float4*>(cs + 2 * e);
        c8[e] = v.x; s8[e] = v.y; c8[e + 1] = v.z; s8[e + 1] = v.w;
    }
}

// 8 rotated pairs (j, j + half) of the projection's values from `at` on
template <bool REDUCE>
__device__ __forceinline__ void rotated_pair(const QkvSource& src, size_t slice, size_t at, int half, const float (&c8)[8],
                                             const float (&s8)[8], float (&o_lo)[8], float (&o_hi)[8]) {
    float lo[8], hi[8];
    if (REDUCE) {
        reduce8_pair(src.partial, src.ksplit, slice, at, half, lo, hi);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            lo[e] = (float)(bf16)lo[e];
            hi[e] = (float)(bf16)hi[e];
        }
    } else {
        load8(src.qkv + at, lo);
        load8(src.qkv + at + half, hi);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        o_lo[e] = lo[e] * c8[e] - hi[e] * s8[e];
        o_hi[e] = hi[e] * c8[e] + lo[e] * s8[e];
    }
}

// One row's queries (rotated, into the projection's buffer) and, for a single new token, its key and value (to the cache):
// thread `u` of the row takes 8 rotation pairs, or 8 values.
template <bool REDUCE>
__device__ __forceinline__ void append_row(const QkvSource& src, const float* __restrict__ tab, const BatchView& bv,
                                           const KvView& kv, int Hq, int seq, int t, bool single, int u) {
    const int d = kv.d, Hkv = kv.Hkv, half = d >> 1, pairs = d >> 4;
    const int nqkv = (Hq + 2 * Hkv) * d;
    const size_t row = (size_t)t * nqkv, slice = (size_t)bv.T * nqkv;
    const int pos = bv.kv_before[seq] + t - bv.q_start[seq];
    const int rotated = (Hq + (single ? Hkv : 0)) * pairs;
    if (u < rotated) {
        const int head = u / pairs, j = (u - head * pairs) * 8;
        float c8[8], s8[8], o_lo[8], o_hi[8];
        load_cos_sin(tab + (size_t)pos * d + 2 * j, c8, s8);
        const size_t at = row + head * d + j;
        rotated_pair<REDUCE>(src, slice, at, half, c8, s8, o_lo, o_hi);
        bf16 *lo = src.qkv + at, *hi = lo + half;
        if (head >= Hq) {
            const int slot = bv.seq_slot[seq];
            bf16* k = kv.k + (size_t)kv.slot_off[slot] * Hkv * d + (size_t)(head - Hq) * kv.slot_cap[slot] * d;
            lo = k + k_piece_offset(pos, j >> 3, d);
            hi = k + k_piece_offset(pos, (half + j) >> 3, d);
        }
        store8(lo, o_lo);
        store8(hi, o_hi);
    } else if (single && u < rotated + Hkv * (d >> 3)) {
        const int head = (u - rotated) / (d >> 3), j = (u - rotated - head * (d >> 3)) * 8;
        float v[8];
        const size_t at = row + (Hq + Hkv + head) * d + j;
        if (REDUCE) reduce8(src.partial, src.ksplit, slice, at, v);
        else load8(src.qkv + at, v);
        const int slot = bv.seq_slot[seq];
        bf16* dst = kv.v + (size_t)kv.slot_off[slot] * Hkv * d + (size_t)head * kv.slot_cap[slot] * d;
#pragma unroll
        for (int e = 0; e < 8; ++e) dst[v_elem_offset(pos, j + e, d)] = (bf16)v[e];
    }
}

// Workgroups from `kv_wgs` on take rows, `row_wgs` each: with partial sums all rows of the batch, else the decode rows.
// `singles`: single new tokens are appended here (otherwise their rows are left alone).
template <bool REDUCE>
__global__ __launch_bounds__(256) void kv_append_kernel(QkvSource src, const float* __restrict__ tab, BatchView bv,
                                                        KvView kv, int Hq, int heads_per_wg, int hgroups, int kv_wgs,
                                                        int row_wgs, int singles) {
    const int d = kv.d, Hkv = kv.Hkv, half = d >> 1;
    const int nqkv = (Hq + 2 * Hkv) * d;
    if ((int)blockIdx.x >= kv_wgs) {
        const int b = blockIdx.x - kv_wgs, r = b / row_wgs;
        const int seq = REDUCE ? bv.token_seq[r] : bv.decode_seqs[r];
        const int t = REDUCE ? r : bv.q_start[seq];
        const bool single = bv.q_start[seq + 1] - bv.q_start[seq] == 1;
        if (single && !singles) return;
        append_row<REDUCE>(src, tab, bv, kv, Hq, seq, t, single, (b - r * row_wgs) * 256 + (int)threadIdx.x);
        return;
    }
    const int item = blockIdx.x / (kAppendBlocks * hgroups);
    const int rest = blockIdx.x - item * (kAppendBlocks * hgroups);
    const int sub = rest / hgroups, hg = rest - sub * hgroups;
    const int s = bv.prefill_items[2 * item], qt = bv.prefill_items[2 * item + 1];
    const int q0 = bv.q_start[s], qlen = bv.q_start[s + 1] - q0;
    if (sub == kAppendBlocks - 1 && (qt + 1) * kPrefillTileQ < qlen) return;
    const int before = bv.kv_before[s], end = before + qlen;
    const int blk = (before >> 5) + qt * 4 + sub;
    const int p_lo = blk * 32 > before ? blk * 32 : before;
    const int p_hi = blk * 32 + 32 < end ? blk * 32 + 32 : end;
    if (p_lo >= p_hi) return;
    const int slot = bv.seq_slot[s];
    const size_t head_stride = (size_t)kv.slot_cap[slot] * d;
    const size_t block_base = (size_t)kv.slot_off[slot] * Hkv * d + (size_t)blk * 32 * d;
    const size_t slice = (size_t)bv.T * nqkv;
    const int tid = threadIdx.x;
    // 256 threads are one head of d = 128 or two of d = 64, in both halves of the kernel
    const int per_head = 2 * d, hsub = tid / per_head, ht = tid - hsub * per_head, n_par = 256 / per_head;
    const int h0 = hg * heads_per_wg + hsub;
    const int h1 = (hg + 1) * heads_per_wg < Hkv ? (hg + 1) * heads_per_wg : Hkv;

    const int uph = d >> 4;                                       // units of 8 pairs (j, j + d/2) per head
    const int p = ht / uph, unit = ht - p * uph;
    const int pos = blk * 32 + p;
    if (pos >= p_lo && pos < p_hi) {
        const size_t row = (size_t)(q0 + pos - before) * nqkv;
        const float* cs = tab + (size_t)pos * d + unit * 16;
        float c8[8], s8[8];
        load_cos_sin(cs, c8, s8);
        for (int h = h0; h < h1; h += n_par) {
            const size_t at = row + (size_t)(Hq + h) * d + unit * 8;
            float o_lo[8], o_hi[8];
            rotated_pair<REDUCE>(src, slice, at, half, c8, s8, o_lo, o_hi);
            bf16* dst = kv.k + block_base + (size_t)h * head_stride + p * 8;
            store8(dst + unit * 256, o_lo);
            store8(dst + (unit + uph) * 256, o_hi);
        }
    }

    const int w = ht / half, j = (ht - w * half) * 2;             // piece of the block, two consecutive head-dim indices
    const int pbase = blk * 32 + 16 * (w >> 1) + 4 * (w & 1);     // the piece holds pbase + {0..3, 8..11}
    const bool whole = pbase >= p_lo && pbase + 11 < p_hi;
    for (int h = h0; h < h1; h += n_par) {
        const size_t col = (size_t)(Hq + Hkv + h) * d + j;
        float a[8], b[8];
        size_t at[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            int pe = pbase + (e & 3) + 8 * (e >> 2);
            pe = pe < p_lo ? p_lo : pe > p_hi - 1 ? p_hi - 1 : pe;            // read in bounds, not stored
            at[e] = (size_t)(q0 + pe - before) * nqkv + col;
            a[e] = b[e] = 0.f;
        }
        if (REDUCE) {
            // two slices' loads of all eight rows go out together (row by row, each waited for the one before)
            for (int k = 0; k < src.ksplit; k += 2) {
                const float* s0 = src.partial + k * slice;
                const float* s1 = k + 1 < src.ksplit ? s0 + slice : s0;
                float2 v[2][8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[0][e] = *reinterpret_cast<const float2*>(s0 + at[e]);
                    v[1][e] = *reinterpret_cast<const float2*>(s1 + at[e]);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    a[e] += v[0][e].x;
                    b[e] += v[0][e].y;
                    if (k + 1 < src.ksplit) {
                        a[e] += v[1][e].x;
                        b[e] += v[1][e].y;
                    }
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bf16x2 v = *reinterpret_cast<const bf16x2*>(src.qkv + at[e]);
                a[e] = (float)v[0];
                b[e] = (float)v[1];
            }
        }
        bf16* dst = kv.v + block_base + (size_t)h * head_stride + ((size_t)w * d + j) * 8;
        if (whole) {
            store8(dst, a);
            store8(dst + 8, b);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int pe = pbase + (e & 3) + 8 * (e >> 2);
                if (pe >= p_lo && pe < p_hi) {
                    dst[e] = (bf16)a[e];
                    dst[8 + e] = (bf16)b[e];
                }
            }
        }
    }
}

bool kv_append_needed(const BatchView& bv, const KvView& kv, int Hq) {
    return bv.n_prefill_items > 0 || (bv.n_decode > 0 && decode_append_apart(bv, kv, Hq));
}
AppendRows kv_append_rows(const QkvSource& src, const BatchView& bv, const KvView& kv, int Hq) {
    const int prompts = bv.T - bv.n_decode, singles = decode_append_apart(bv, kv, Hq) ? bv.n_decode : 0;
    return AppendRows{prompts + singles, (src.partial ? prompts : 0) + singles};
}

void launch_kv_append(const QkvSource& src, const float* rope_tab, const BatchView& bv, const KvView& kv, int Hq,
                      hipStream_t st) {
    if (!kv_append_needed(bv, kv, Hq)) return;
    const int blocks = bv.n_prefill_items * kAppendBlocks;
    const int n_par = 128 / kv.d;                      // heads that run side by side in a workgroup
    // Several heads per workgroup share the load of cosines and sines, as long as some thousand workgroups remain: 14 091
    // rows of 40 heads 126 us with one head each, 109 with five; 4973 rows of 32 heads 41.7 and 41.5 either way.
    int hpw = (int)((int64_t)blocks * kv.Hkv / 4096);
    hpw = hpw < n_par ? n_par : hpw > 8 ? 8 : hpw;
    const int hgroups = (kv.Hkv + hpw - 1) / hpw;
    const bool singles = bv.n_decode > 0 && decode_append_apart(bv, kv, Hq);
    // threads per row: rotation pairs by eights, and a single new token's values by eights
    const int units = (Hq + (singles ? kv.Hkv : 0)) * (kv.d >> 4) + (singles ? kv.Hkv * (kv.d >> 3) : 0);
    const int kv_wgs = blocks * hgroups, row_wgs = (units + 255) / 256;
    const int rows = src.partial ? bv.T : singles ? bv.n_decode : 0;
    auto kern = src.partial ? kv_append_kernel<true> : kv_append_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(kv_wgs + rows * row_wgs), dim3(256), 0, st, src, rope_tab, bv, kv, Hq, hpw, hgroups, kv_wgs,
                       row_wgs, (int)singles);
}

#else  // BZ_FP32_DEBUG: one workgroup per token rotates its queries in place, and its keys into the cache, and copies its values

__global__ __launch_bounds__(256) void rope_append_kernel(float* __restrict__ qkv, const float* __restrict__ tab, BatchView bv,
                                                          KvView kv, int Hq) {
    const int d = kv.d, Hkv = kv.Hkv, half = d >> 1;
    const int t = blockIdx.x, s = bv.token_seq[t];
    const int pos = bv.kv_before[s] + (t - bv.q_start[s]);
    const int slot = bv.seq_slot[s];
    const size_t head_stride = (size_t)kv.slot_cap[slot] * d;
    const size_t slot_base = (size_t)kv.slot_off[slot] * Hkv * d;
    float* row = qkv + (size_t)t * (Hq + 2 * Hkv) * d;
    const float* cs = tab + (size_t)pos * d;
    for (int u = threadIdx.x; u < (Hq + Hkv) * half; u += 256) {
        const int head = u / half, j = u - head * half;
        const float lo = row[head * d + j], hi = row[head * d + half + j];
        const float c = cs[2 * j], sn = cs[2 * j + 1];
        const float o_lo = lo * c - hi * sn, o_hi = hi * c + lo * sn;
        if (head < Hq) {
            row[head * d + j] = o_lo;
            row[head * d + half + j] = o_hi;
        } else {
            float* dst = kv.k + slot_base + (size_t)(head - Hq) * head_stride;
            dst[k_elem_offset(pos, j, d)] = o_lo;
            dst[k_elem_offset(pos, half + j, d)] = o_hi;
        }
    }
    for (int u = threadIdx.x; u < Hkv * d; u += 256)
        kv.v[slot_base + (size_t)(u / d) * head_stride + v_elem_offset(pos, u % d, d)] = row[(Hq + Hkv) * d + u];
}

bool kv_append_needed(const BatchView& bv, const KvView&, int) { return bv.T > 0; }
AppendRows kv_append_rows(const QkvSource&, const BatchView& bv, const KvView&, int) { return AppendRows{bv.T, bv.T}; }

void launch_kv_append(const QkvSource& src, const float* rope_tab, const BatchView& bv, const KvView& kv, int Hq,
                      hipStream_t st) {
    if (bv.T <= 0) return;
    hipLaunchKernelGGL(rope_append_kernel, dim3(bv.T), dim3(256), 0, st, src.qkv, rope_tab, bv, kv, Hq);
}
#endif

// ---------------------------------------------------------------------------------------------
// KV scatter/gather between token-major [n, Hkv, d] buffers and the cache layout of one slot.
// K: one thread per 8 head-dim elements of a token (16 bytes on both sides).  V: one thread per
// (piece of 8 positions, kv head, j), 16 bytes on the cache side; pieces that the range
// [pos0, pos0 + n) covers only partly are handled element by element.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void kv_scatter_kernel(const act_t* __restrict__ src_k,
                                                         const act_t* __restrict__ src_v, KvView kv, int slot,
                                                         int pos0, int n, int to_cache,
                                                         act_t* __restrict__ dst_k, act_t* __restrict__ dst_v) {
    const int d = kv.d, Hkv = kv.Hkv;
    const int cap = kv.slot_cap[slot];
    const size_t slot_base = (size_t)kv.slot_off[slot] * Hkv * d;
    const int vec_per_tok = Hkv * (d >> 3);
    const size_t k_total = (size_t)n * vec_per_tok;
    const int piece0 = (pos0 >> 5) * 4;                          // first piece of the first block touched
    const int n_pieces = (((pos0 + n - 1) >> 5) + 1) * 4 - piece0;
    const size_t v_total = (size_t)n_pieces * Hkv * d;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < k_total + v_total;
         i += (size_t)gridDim.x * blockDim.x) {
        if (i < k_total) {
            const int tok = (int)(i / vec_per_tok);
            const int w = (int)(i - (size_t)tok * vec_per_tok);
            const int kvh = w / (d >> 3);
            const int j0 = (w - kvh * (d >> 3)) * 8;
            const size_t lin = (size_t)tok * Hkv * d + (size_t)kvh * d + j0;
            const size_t cac_k = slot_base + (size_t)kvh * cap * d + k_piece_offset(pos0 + tok, j0 >> 3, d);
            float a[8];
            if (to_cache) {
                load8(src_k + lin, a);
                store8(kv.k + cac_k, a);
            } else {
                load8(kv.k + cac_k, a);
                store8(dst_k + lin, a);
            }
        } else {
            const size_t vi = i - k_total;
            const int u = (int)(vi % ((size_t)Hkv * d));          // kvh * d + j: consecutive lanes, consecutive j
            const int piece = piece0 + (int)(vi / ((size_t)Hkv * d));
            const int kvh = u / d, j = u - kvh * d;
            const int w = piece & 3;                              // piece 2t + h of its block
            const int pbase = (piece >> 2) * 32 + 16 * (w >> 1) + 4 * (w & 1);
            act_t* cv = kv.v + slot_base + (size_t)kvh * cap * d + (size_t)(piece >> 2) * 32 * d + ((size_t)w * d + j) * 8;
            const bool whole = pbase >= pos0 && pbase + 11 < pos0 + n;
            if (to_cache) {
                if (whole) {
                    float b[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        b[e] = to_f32(src_v[(size_t)(pbase + (e & 3) + 8 * (e >> 2) - pos0) * Hkv * d + u]);
                    store8(cv, b);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int p = pbase + (e & 3) + 8 * (e >> 2);
                        if (p >= pos0 && p < pos0 + n) cv[e] = src_v[(size_t)(p - pos0) * Hkv * d + u];
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int p = pbase + (e & 3) + 8 * (e >> 2);
                    if (p >= pos0 && p < pos0 + n) dst_v[(size_t)(p - pos0) * Hkv * d + u] = cv[e];
                }
            }
        }
    }
}

void launch_kv_scatter(const act_t* src_k, const act_t* src_v, const KvView& kv, int slot, int pos0, int n,
                       bool to_cache, act_t* dst_k, act_t* dst_v, hipStream_t st) {
    if (n <= 0) return;
    const size_t n_pieces = (size_t)((((pos0 + n - 1) >> 5) + 1) - (pos0 >> 5)) * 4;
    const size_t total = (size_t)n * kv.Hkv * (kv.d >> 3) + n_pieces * kv.Hkv * kv.d;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(kv_scatter_kernel, dim3(blocks), dim3(256), 0, st, src_k, src_v, kv, slot, pos0, n,
                       to_cache ? 1 : 0, dst_k, dst_v);
}

// One workgroup: moves every sequence one position on, then lists the (sequence, chunk) pairs the decode
// attention has to visit at the new lengths, sequence by sequence (an exclusive scan over chunk counts).
__global__ __launch_bounds__(256) void batch_advance_kernel(int32_t* kv_before, int B, const int32_t* __restrict__ decode_seqs,
                                                            const int32_t* __restrict__ seq_slot, int n_decode, int4* work,
                                                            int capacity) {
    __shared__ int scan[256];
    __shared__ int base;
    const int tid = threadIdx.x;
    for (int i = tid; i < B; i += 256) kv_before[i] += 1;
    if (tid == 0) base = 0;
    __syncthreads();
    for (int d0 = 0; d0 < n_decode; d0 += 256) {
        const int di = d0 + tid;
        int s = 0, n = 0;
        if (di < n_decode) {
            s = decode_seqs[di];
            n = (kv_before[s] + 1 + kDecodeChunk - 1) / kDecodeChunk;
        }
        scan[tid] = n;
        __syncthreads();
        for (int step = 1; step < 256; step <<= 1) {
            const int add = tid >= step ? scan[tid - step] : 0;
            __syncthreads();
            scan[tid] += add;
            __syncthreads();
        }
        const int at = base + scan[tid] - n;
        if (n > 0) {
            const int slot = seq_slot[s];
            for (int c = 0; c < n; ++c)
                if (at + c < capacity) {
                    work[2 * (at + c)] = make_int4(s, slot, di, n);
                    work[2 * (at + c) + 1] = make_int4(at, 0, 0, 0);
                }
        }
        __syncthreads();
        if (tid == 255) base += scan[255];
        __syncthreads();
    }
}

// Slot table entry of one KV slot, written in stream order (a host-to-device copy of four bytes would
// block the calling thread).
__global__ void set_slot_kernel(int32_t* off, int32_t* cap, int32_t off_v, int32_t cap_v) {
    if (threadIdx.x == 0) {
        *off = off_v;
        *cap = cap_v;
    }
}

void launch_set_slot(int32_t* off, int32_t* cap, int32_t off_v, int32_t cap_v, hipStream_t st) {
    hipLaunchKernelGGL(set_slot_kernel, dim3(1), dim3(64), 0, st, off, cap, off_v, cap_v);
}

void launch_batch_advance(int32_t* kv_before, int B, const int32_t* decode_seqs, const int32_t* seq_slot, int n_decode,
                          int4* work, int capacity, hipStream_t st) {
    hipLaunchKernelGGL(batch_advance_kernel, dim3(1), dim3(256), 0, st, kv_before, B, decode_seqs, seq_slot, n_decode, work,
                       capacity);
}

}  // namespace bz
