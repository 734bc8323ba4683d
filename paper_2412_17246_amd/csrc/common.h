// Internal definitions shared by the library's host code and kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "blitz_layer.h"

namespace bz {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Activation element: bf16 in the product build, float in the fp32 debug build.
#ifdef BZ_FP32_DEBUG
typedef float act_t;
#else
typedef bf16 act_t;
#endif

constexpr int kWave = 64;

// A kernel's dynamic-LDS limit is a per-function, per-device setting.  One of these per kernel
// instantiation remembers on which devices the limit has been raised (or refused), so that the call is
// made once per device; threads that race here make the same idempotent call.  A refusal is consumed
// here and reported as false, never by a later HIP call.
struct LdsLimit {
    std::atomic<uint64_t> granted{0}, refused{0};
    bool raise(const void* fn, int bytes) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        const uint64_t bit = (dev >= 0 && dev < 64) ? (uint64_t)1 << dev : 0;    // devices past 63: asked every time
        if (granted.load(std::memory_order_acquire) & bit) return true;
        if (refused.load(std::memory_order_acquire) & bit) return false;
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) {
            (void)hipGetLastError();
            refused.fetch_or(bit, std::memory_order_release);
            return false;
        }
        granted.fetch_or(bit, std::memory_order_release);
        return true;
    }
};

// ---- 8-element loads / stores, converting to and from float --------------------------------
__device__ __forceinline__ void load8(const bf16* p, float (&v)[8]) {
    bf16x8 t = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (float)t[i];
}
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
    float4 a = reinterpret_cast<const float4*>(p)[0];
    float4 b = reinterpret_cast<const float4*>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void store8(bf16* p, const float (&v)[8]) {
    bf16x8 t;
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = (bf16)v[i];
    *reinterpret_cast<bf16x8*>(p) = t;
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
    reinterpret_cast<float4*>(p)[0] = make_float4(v[0], v[1], v[2], v[3]);
    reinterpret_cast<float4*>(p)[1] = make_float4(v[4], v[5], v[6], v[7]);
}
// 8 activation elements kept in their storage format (so loads in flight cost few registers)
struct raw8_bf16 { bf16x8 v; };
struct raw8_f32 { float4 a, b; };
__device__ __forceinline__ void load_raw8(const bf16* p, raw8_bf16& r) { r.v = *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ void load_raw8(const float* p, raw8_f32& r) {
    r.a = reinterpret_cast<const float4*>(p)[0];
    r.b = reinterpret_cast<const float4*>(p)[1];
}
__device__ __forceinline__ float raw_get(const raw8_bf16& r, int e) { return (float)r.v[e]; }
__device__ __forceinline__ float raw_get(const raw8_f32& r, int e) {
    return e == 0 ? r.a.x : e == 1 ? r.a.y : e == 2 ? r.a.z : e == 3 ? r.a.w
         : e == 4 ? r.b.x : e == 5 ? r.b.y : e == 6 ? r.b.z : r.b.w;
}
#ifdef BZ_FP32_DEBUG
typedef raw8_f32 raw8_act;
#else
typedef raw8_bf16 raw8_act;
#endif

__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ void from_f32(bf16& o, float v) { o = (bf16)v; }
__device__ __forceinline__ void from_f32(float& o, float v) { o = v; }

// sum over split-K slices, in slice order, of 8 consecutive partial sums of row m.  Loads go out four
// slices at a time (a slice index past the end re-reads the last slice; its value is not added).
__device__ __forceinline__ void reduce8(const float* __restrict__ partial, int ksplit, size_t slice_stride,
                                        size_t off, float (&s)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = 0.f;
    for (int k0 = 0; k0 < ksplit; k0 += 4) {
        float4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = (k0 + u < ksplit) ? k0 + u : ksplit - 1;
            a[u] = *reinterpret_cast<const float4*>(partial + k * slice_stride + off);
            b[u] = *reinterpret_cast<const float4*>(partial + k * slice_stride + off + 4);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + u < ksplit) {
                s[0] += a[u].x; s[1] += a[u].y; s[2] += a[u].z; s[3] += a[u].w;
                s[4] += b[u].x; s[5] += b[u].y; s[6] += b[u].z; s[7] += b[u].w;
            }
    }
}

// The same for the two halves of a rotation, `half` values apart, whose loads go out together.
__device__ __forceinline__ void reduce8_pair(const float* __restrict__ partial, int ksplit, size_t slice_stride, size_t off,
                                             int half, float (&lo)[8], float (&hi)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) lo[e] = hi[e] = 0.f;
    for (int k0 = 0; k0 < ksplit; k0 += 4) {
        float4 v[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float* p = partial + (k0 + u < ksplit ? k0 + u : ksplit - 1) * slice_stride + off;
            v[u][0] = *reinterpret_cast<const float4*>(p);
            v[u][1] = *reinterpret_cast<const float4*>(p + 4);
            v[u][2] = *reinterpret_cast<const float4*>(p + half);
            v[u][3] = *reinterpret_cast<const float4*>(p + half + 4);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + u < ksplit) {
                lo[0] += v[u][0].x; lo[1] += v[u][0].y; lo[2] += v[u][0].z; lo[3] += v[u][0].w;
                lo[4] += v[u][1].x; lo[5] += v[u][1].y; lo[6] += v[u][1].z; lo[7] += v[u][1].w;
                hi[0] += v[u][2].x; hi[1] += v[u][2].y; hi[2] += v[u][2].z; hi[3] += v[u][2].w;
                hi[4] += v[u][3].x; hi[5] += v[u][3].y; hi[6] += v[u][3].z; hi[7] += v[u][3].w;
            }
    }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

// silu(z) = z / (1 + exp(-z)) with the hardware's exponential and reciprocal (about 1 ulp each; every
// use rounds the product to bf16 afterwards).  An IEEE division costs ten instructions per element in the
// epilogue of the gate/up projection, which has 128 of them per lane and tile.  One definition for every
// kernel that applies SwiGLU, so that they agree bit for bit.
__device__ __forceinline__ float silu_fast(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// Device-side view of the KV cache of one layer.  K part then V part; inside a part, slot s
// starts at element slot_off[s] * Hkv * d and holds Hkv heads of slot_cap[s] positions each
// (slot_cap is a multiple of 32).  Both K and V of one head are stored in blocks of 32 positions,
// each block (32 * d elements, contiguous) in the order in which a 32x32x16 MFMA wants its row
// operand, so attention reads the cache as it lies in memory with 16-byte loads:
//   K (row = position, contraction over d): the 8-element pieces of the head vector are stored
//   piece-major: element (pos, j) lies at k_elem_offset(pos, j, d).  A wave reading piece c of 32
//   consecutive positions touches 512 contiguous bytes.
//   V (row = head dim, contraction over positions): 8 positions form a piece, pieces are stored
//   [piece][j][8].  The 8 positions of piece w = 2t + h are {16t + 4h + 0..3, 16t + 8 + 4h + 0..3}:
//   exactly the positions that lane half h of a 32x32 accumulator holds for k-step t, so softmax
//   probabilities go from the score accumulators into the second MFMA without leaving registers.
__host__ __device__ inline size_t k_piece_offset(int pos, int piece, int d) {
    return (size_t)(pos >> 5) * 32 * d + (((size_t)piece * 32 + (pos & 31)) << 3);
}
__host__ __device__ inline size_t k_elem_offset(int pos, int j, int d) { return k_piece_offset(pos, j >> 3, d) + (j & 7); }
__host__ __device__ inline size_t v_elem_offset(int pos, int j, int d) {
    const int p = pos & 31, t = p >> 4, g = p & 15, h = (g >> 2) & 1, e = (g & 3) + ((g >> 3) << 2);
    return (size_t)(pos >> 5) * 32 * d + (((size_t)(2 * t + h) * d + j) << 3) + e;
}

struct KvView {
    act_t* k;                 // layer's K part
    act_t* v;                 // layer's V part
    const int32_t* slot_off;  // [max_seqs] first token of the slot inside the arena
    const int32_t* slot_cap;  // [max_seqs] capacity in tokens
    int Hkv;
    int d;
};

// Device-side view of a batch.
struct BatchView {
    int B;
    int T;
    const int32_t* q_start;     // [B+1]
    const int32_t* seq_slot;    // [B]
    const int32_t* kv_before;   // [B]
    const int32_t* token_seq;   // [T] sequence index of each packed row
    const int32_t* prefill_items;  // [n_prefill_items][2] = (seq, q_tile)
    int n_prefill_items;
    int prefill_keys;              // longest key range of a prefill item
    const int32_t* decode_seqs;    // [n_decode] sequence indices with exactly one new token
    int n_decode;
    int decode_chunks;             // upper bound on ceil((kv_before+1)/kDecodeChunk) over decode seqs
    // One entry (two int4) per (decode sequence, chunk of its cache) that exists now, sequence by
    // sequence: (sequence index, KV slot, index into decode_seqs, chunks of this sequence), (index of
    // the sequence's first entry, 0, 0, 0).  The decode attention runs n_decode_work * Hkv workgroups;
    // workgroup b reads entry b / Hkv, which belongs to the right sequence, and takes
    // (kv head, chunk) = divmod(b - Hkv * first, chunks): a sequence's kv heads one after the other,
    // each head's chunks in order, which is the order the cache lies in memory.
    const int4* decode_work;
    int n_decode_work;
};

// The QKV projection of a batch, rows of (Hq + 2 Hkv) * d values: query, key and value heads.  Either the projection's
// output (`partial` null) or its split-K partial sums partial[ksplit][T][row], which the reader adds in slice order and
// rounds to the activation type, as the GEMM's own epilogue would have.
struct QkvSource {
    act_t* qkv;
    const float* partial;
    int ksplit;
};

constexpr int kPrefillTileQ = 128;   // query rows per prefill-attention workgroup
constexpr int kDecodeChunk = 256;    // KV positions per decode-attention workgroup

// ---- launchers (each enqueues on `st`; shapes are validated by the callers) ------------------
void launch_rmsnorm(const act_t* x, const bf16* gain, act_t* y, int T, int H, float eps, hipStream_t st);
// `ws` is fp32 scratch, best of at least gemm_workspace_bytes(mode, M, N, K) bytes (0 for shapes that need none).  With less,
// K is cut into fewer ranges, or a kernel that needs no scratch takes the problem.
void launch_gemm(int mode, const act_t* a, const bf16* w, const act_t* r, act_t* c, int M, int N, int K,
                 float* ws, size_t ws_bytes, hipStream_t st);
size_t gemm_workspace_bytes(int mode, int M, int N, int K);
size_t gemm_instance_bytes(int mode, int M, int N, int K);      // what an instance sets aside for the problem
void gemm_plan(int mode, int M, int N, int K, size_t room, bz_gemm_plan* out);
// Problems whose plan cuts K only: computes the split-K partial sums partial[ksplit][M][Nrows] (Nrows = 2N
// in SwiGLU mode) into `ws` and returns ksplit, leaving the slice-order reduction and the epilogue
// to the consumer kernel; returns 0 (and does nothing) when the shape does not take that path.
int launch_gemm_partial(int mode, const act_t* a, const bf16* w, int M, int N, int K, float* ws, size_t ws_bytes,
                        hipStream_t st);
// x[T,H] += sum over slices of partial[k][T][H] (slice order), rounded to the activation type and
// stored; then, unless gain is null, y = rmsnorm(x) * gain exactly as launch_rmsnorm would compute it.
void launch_reduce_residual_rmsnorm(act_t* x, const float* partial, int ksplit, const bf16* gain, act_t* y, int T,
                                    int H, float eps, hipStream_t st);
// Rotary embedding (table `rope_tab`: [max_seq_len][d/2] pairs of cos, sin) and the append to the cache are shared out so
// that the projection is read once and the rotated queries never travel through memory: launch_kv_append takes the keys
// and values of the sequences with several new tokens, the prefill kernel rotates its queries as it loads them, and the
// decode kernel does both for its one token per sequence (below a number of workgroups).  Where the projection is partial sums, launch_kv_append also folds
// and rotates the queries of those sequences into `qkv`: in the prefill kernel every lane would fold a row of its own, line by
// line.  (fp32 debug build: launch_kv_append does it all.)  launch_kv_append comes first.
bool kv_append_needed(const BatchView& bv, const KvView& kv, int Hq);
// Whether single new tokens are rotated and appended by launch_kv_append as well.  Inside the decode kernel that costs every
// workgroup 0.4 us and more of its 9 to 10, a launch of its own 6 to 10 us altogether: on grids of many workgroups it is the
// cheaper.  Attention with the append, inside against apart, us: one query head per kv head 171.5 / 173.5 (8.8 thousand
// workgroups), 212 / 209 (10.9), 308 / 301 (15.9), 392 / 386 (20); two 408 / 403 (20); four 367 / 371 (16).  Batches of mostly
// one chunk per sequence stay inside, where they need no combine (10 thousand workgroups: 169 / 183).
inline bool decode_append_apart(const BatchView& bv, const KvView& kv, int Hq) {
    return bv.n_decode_work >= 2 * bv.n_decode && (int64_t)bv.n_decode_work * kv.Hkv > 9600 * (int64_t)(Hq / kv.Hkv);
}
// rows whose keys and values, and rows whose queries, launch_kv_append takes
struct AppendRows { int kv, q; };
AppendRows kv_append_rows(const QkvSource& src, const BatchView& bv, const KvView& kv, int Hq);
void launch_kv_append(const QkvSource& src, const float* rope_tab, const BatchView& bv, const KvView& kv, int Hq,
                      hipStream_t st);
void launch_attn_prefill(const QkvSource& src, const float* rope_tab, act_t* out, const BatchView& bv, const KvView& kv,
                         int Hq, hipStream_t st);
// combine: false where the caller combines the chunks itself (few_combines); then a single chunk leaves partial results, too
void launch_attn_decode(const QkvSource& src, const float* rope_tab, act_t* out, float* partial, const BatchView& bv,
                        const KvView& kv, int Hq, bool combine, hipStream_t st);
// Few rows: the projections with everything around them in one launch each.  mode 0: c = rmsnorm(x) * gain * w^T; 1: c = r +
// x * w^T (r may be c); 2: c = silu(gate) * up of rmsnorm(x) * gain.  For the batches that few_rows names.
void launch_few(int mode, const act_t* x, const bf16* gain, float eps, const bf16* w, const act_t* r, act_t* c, int M, int N,
                int K, hipStream_t st);
// The output projection of single new tokens whose attention left partial results (no combine launch then): x += combined * w^T.
bool few_combines(const BatchView& bv, int qd);
void launch_few_out(const float* partial, const BatchView& bv, const KvView& kv, const bf16* w, act_t* x, int H, int qd, hipStream_t st);
void launch_kv_scatter(const act_t* src_k, const act_t* src_v, const KvView& kv, int slot, int pos0, int n,
                       bool to_cache, act_t* dst_k, act_t* dst_v, hipStream_t st);
// kv_before[s] += 1 for every sequence, then the decode work list is rebuilt for the new lengths
// (at most `capacity` entries are written; the caller has checked that they suffice)
void launch_batch_advance(int32_t* kv_before, int B, const int32_t* decode_seqs, const int32_t* seq_slot, int n_decode,
                          int4* work, int capacity, hipStream_t st);

void launch_set_slot(int32_t* off, int32_t* cap, int32_t off_v, int32_t cap_v, hipStream_t st);

// floats per (decode sequence, query head, chunk) in the decode partial buffer: d outputs, max, sum
__host__ __device__ inline int decode_partial_stride(int d) { return d + 2; }

}  // namespace bz
