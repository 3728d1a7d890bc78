// Server-side scatter (Algorithm 2, "M <- M - decode(g)"), worker apply, index validation,
// the wire form of a message, and the pull without secondary compression.
#include "dgs_wave.h"

namespace dgs {

// ---------------------------------------------------------------------------
// sparse scatter: push, apply, validation
// ---------------------------------------------------------------------------

// blockIdx.y selects the destination buffer (model first, then the difference
// rows), so a wavefront walks ascending indices of one buffer.  Indices are
// unique within a message, and calls are ordered on one stream: no atomics.
__global__ __launch_bounds__(256) void k_push(float *model, float *diff, uint32_t n,
                                              const uint32_t *idx, const float *val, uint32_t nnz,
                                              uint32_t first_buf)
{
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= nnz) return;
    const uint32_t b = blockIdx.y + first_buf;
    float *dst = (b == 0) ? model : diff + (size_t)(b - 1) * n;
    const uint32_t i = idx[e];
    if (i < n) store_scattered(&dst[i], dst[i] - val[e]);
}

void launch_push(float *model, float *diff, uint32_t W, uint32_t n, const uint32_t *idx,
                 const float *val, uint32_t nnz, void *stream, void *ev0, void *ev1)
{
    if (nnz == 0) return;
    const uint32_t first = model ? 0u : 1u;
    const uint32_t bufs = W + 1 - first;
    if (bufs == 0) return;
    // gridDim.y is limited to 65535: loop over slabs of buffers
    for (uint32_t b0 = 0; b0 < bufs; b0 += 32768) {
        const uint32_t nb = (bufs - b0 < 32768u) ? (bufs - b0) : 32768u;
        // events time the first slab only (one slab unless there are more than 32768 buffers)
        launch_k(k_push, dim3((nnz + 255) / 256, nb), dim3(256), (hipStream_t)stream,
                 b0 == 0 ? ev0 : nullptr, b0 == 0 ? ev1 : nullptr, model, diff, n, idx, val, nnz,
                 first + b0);
    }
}

__global__ __launch_bounds__(256) void k_validate_idx(const uint32_t *idx, uint32_t nnz, uint32_t n,
                                                      uint32_t *flag)
{
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= nnz) return;
    const uint32_t i = idx[e];
    bool bad = (i >= n);
    if (e > 0 && idx[e - 1] >= i) bad = true;
    if (bad) atomicOr(flag, 1u);
}

void launch_validate_idx(const uint32_t *idx, uint32_t nnz, uint32_t n, uint32_t *flag, void *stream)
{
    if (nnz == 0) return;
    hipLaunchKernelGGL(k_validate_idx, dim3((nnz + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       idx, nnz, n, flag);
}

// An index outside [0, n) is skipped, as in k_push: a corrupted message must not write
// outside the destination.
__global__ __launch_bounds__(256) void k_apply(float *dst, uint32_t n, const uint32_t *idx, const float *val,
                                               uint32_t nnz, float sign)
{
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= nnz) return;
    const uint32_t i = idx[e];
    if (i < n) dst[i] = __builtin_fmaf(sign, val[e], dst[i]);
}

void launch_apply(float *dst, uint32_t n, const uint32_t *idx, const float *val, uint32_t nnz, float sign,
                  void *stream)
{
    if (nnz == 0) return;
    hipLaunchKernelGGL(k_apply, dim3((nnz + 255) / 256), dim3(256), 0, (hipStream_t)stream, dst, n, idx,
                       val, nnz, sign);
}

// ---------------------------------------------------------------------------
// wire form of a message: fp32 values, then per tensor its local indices bit-packed
// ---------------------------------------------------------------------------

// Last tensor whose `field` (ascending over the tensors) is <= x.
template <uint32_t PlanEntry::*FIELD>
__device__ __forceinline__ uint32_t plan_search(const PlanEntry *plan, uint32_t J, uint32_t x)
{
    uint32_t lo = 0, hi = J;                 // invariant: plan[lo].FIELD <= x, answer in [lo, hi)
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (plan[mid].*FIELD <= x) lo = mid; else hi = mid;
    }
    return lo;                               // offsets increase strictly: every tensor has k_j >= 1
}

// binary32 -> bfloat16 (its upper half), to nearest, halfway cases to the even one; beyond the
// largest finite bfloat16 the carry runs into the exponent and gives infinity; NaN stays NaN.
__device__ __forceinline__ uint32_t to_bf16(float x)
{
    const uint32_t b = __float_as_uint(x);
    if ((b << 1) > 0xFF000000u) return (b >> 16) | 0x40u;
    return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}

// Words of the value area: one per fp32 value, or one per two bfloat16 values.
__host__ __device__ __forceinline__ uint32_t wire_value_words(uint32_t K, uint32_t value_bits)
{
    return value_bits == 16u ? (K + 1u) / 2u : K;
}

// One thread per word of the value area (a copied fp32 value, or two values rounded to bfloat16)
// and per 32-bit word of the index area: the word gathers the pieces of the entries that overlap
// it (entry e of tensor j covers bits [e b_j, (e + 1) b_j) of the tensor's block).  Out-of-tensor
// indices are masked to b_j bits and, with `flag`, reported.
__global__ __launch_bounds__(256) void k_wire_pack(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t J,
                                                   uint32_t K, uint32_t words, uint32_t value_bits,
                                                   const uint32_t *idx, const float *val, uint32_t *wire,
                                                   uint32_t *flag)
{
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint32_t vw = wire_value_words(K, value_bits);
    if (t < vw) {
        if (value_bits == 16u) {
            const uint32_t e = 2u * (uint32_t)t;
            wire[t] = to_bf16(val[e]) | ((e + 1u < K) ? (to_bf16(val[e + 1u]) << 16) : 0u);
        } else {
            wire[t] = __float_as_uint(val[t]);
        }
        return;
    }
    if (t >= (uint64_t)vw + words) return;
    const uint32_t w = (uint32_t)(t - vw);
    const uint32_t j = plan_search<&PlanEntry::wire_off>(plan, J, w);
    const PlanEntry pe = plan[j];
    const TensorDesc td = tdesc[j];
    const uint32_t b = pe.wire_bits;
    const uint64_t bit0 = (uint64_t)(w - pe.wire_off) * 32u;           // first bit of this word in the block
    const uint64_t e0 = bit0 / b;
    if (e0 >= pe.k) { wire[t] = 0; return; }                           // cannot happen: blocks end with their last entry
    const uint64_t e1 = min((uint64_t)pe.k - 1u, (bit0 + 31u) / b);
    const uint32_t mask = (b >= 32u) ? 0xFFFFFFFFu : ((1u << b) - 1u);
    uint32_t word = 0;
    bool bad = false;
    for (uint64_t e = e0; e <= e1; ++e) {
        const uint32_t local = idx[pe.outoff + e] - td.off;
        bad |= local >= td.n;
        const uint64_t pos = e * b;
        const uint32_t piece = local & mask;
        word |= (pos >= bit0) ? (piece << (uint32_t)(pos - bit0)) : (piece >> (uint32_t)(bit0 - pos));
    }
    wire[t] = word;
    if (bad && flag) atomicOr(flag, 1u);
}

// One thread per entry: value copied (a bfloat16 widened), local index cut out of one or two
// words of its block.
__global__ __launch_bounds__(256) void k_wire_unpack(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t J,
                                                     uint32_t K, uint32_t value_bits, const uint32_t *wire,
                                                     uint32_t *idx, float *val, uint32_t *flag)
{
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= K) return;
    if (value_bits == 16u) {
        const uint32_t w2 = wire[t >> 1];
        val[t] = __uint_as_float((t & 1u) ? (w2 & 0xFFFF0000u) : (w2 << 16));
    } else {
        val[t] = __uint_as_float(wire[t]);
    }
    const uint32_t j = plan_search<&PlanEntry::outoff>(plan, J, (uint32_t)t);
    const PlanEntry pe = plan[j];
    const TensorDesc td = tdesc[j];
    const uint32_t b = pe.wire_bits;
    const uint64_t pos = (uint64_t)((uint32_t)t - pe.outoff) * b;
    const uint32_t *block = wire + wire_value_words(K, value_bits) + pe.wire_off;
    const uint32_t w = (uint32_t)(pos >> 5), sh = (uint32_t)(pos & 31u);
    uint64_t x = block[w];
    if (sh + b > 32u) x |= (uint64_t)block[w + 1] << 32;              // an entry that crosses ends inside the block
    const uint32_t mask = (b >= 32u) ? 0xFFFFFFFFu : ((1u << b) - 1u);
    const uint32_t local = (uint32_t)(x >> sh) & mask;
    idx[t] = td.off + local;
    if (local >= td.n && flag) atomicOr(flag, 1u);
}

void launch_wire_pack(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t J, uint32_t K, uint32_t words,
                      uint32_t value_bits, const uint32_t *idx, const float *val, uint32_t *wire, uint32_t *flag,
                      void *stream, void *ev0, void *ev1)
{
    const uint64_t threads = (uint64_t)wire_value_words(K, value_bits) + words;
    if (threads == 0) return;
    launch_k(k_wire_pack, dim3((uint32_t)((threads + 255) / 256)), dim3(256), (hipStream_t)stream, ev0, ev1,
             tdesc, plan, J, K, words, value_bits, idx, val, wire, flag);
}

void launch_wire_unpack(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t J, uint32_t K,
                        uint32_t value_bits, const uint32_t *wire, uint32_t *idx, float *val, uint32_t *flag,
                        void *stream, void *ev0, void *ev1)
{
    if (K == 0) return;
    launch_k(k_wire_unpack, dim3((K + 255) / 256), dim3(256), (hipStream_t)stream, ev0, ev1, tdesc, plan, J, K,
             value_bits, wire, idx, val, flag);
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t *p, uint32_t v, size_t count)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * 256;
    for (; i < count; i += stride) p[i] = v;
}

void launch_fill_u32(uint32_t *p, uint32_t v, size_t count, void *stream)
{
    if (count == 0) return;
    size_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)blocks), dim3(256), 0, (hipStream_t)stream, p, v, count);
}

// A small host table carried to the device inside kernel arguments (no copy engine, no
// staging buffer): PUT_WORDS 32-bit words per launch.
constexpr uint32_t PUT_WORDS = 768;
struct PutChunk { uint32_t w[PUT_WORDS]; };

__global__ __launch_bounds__(256) void k_put_words(uint32_t *dst, const PutChunk c, uint32_t count)
{
    for (uint32_t i = threadIdx.x; i < count; i += 256) dst[i] = c.w[i];
}

void launch_put_words(uint32_t *dst, const uint32_t *src_host, size_t words, void *stream)
{
    for (size_t o = 0; o < words; o += PUT_WORDS) {
        PutChunk c;
        const uint32_t cnt = (uint32_t)((words - o < PUT_WORDS) ? (words - o) : PUT_WORDS);
        for (uint32_t i = 0; i < cnt; ++i) c.w[i] = src_host[o + i];
        for (uint32_t i = cnt; i < PUT_WORDS; ++i) c.w[i] = 0;
        hipLaunchKernelGGL(k_put_words, dim3(1), dim3(256), 0, (hipStream_t)stream, dst + o, c, cnt);
    }
}

// ---------------------------------------------------------------------------
// pull without secondary compression: every nonzero of one difference row, or of
// model - sent_k when a model is given (the server state as Algorithm 2 prints it)
// ---------------------------------------------------------------------------
//
// count  one wavefront per tile reads the row once (bound by that read), counts the nonzeros and
//        leaves them, in order, in the tile's slots as long as they fit (a quarter of the tile)
// scan   one workgroup per PULL_CHUNK tiles: list positions inside the chunk; the last one to
//        finish adds the chunks up and hands the total to the host
// emit   copies the lists to their place and settles the row; only a tile that outgrew its slots
//        is read again.  Does nothing if the total exceeds the caller's capacity.
// 108M parameters, 2 % nonzero: 78 + 7 + 73 us, the emission bound by its scattered 4-byte stores
// (element-wise loads in both passes and a scan by one workgroup: 118 + 189 + 135 us, and 35 us in
// which the GPU waited for the host to see the count).

__device__ __forceinline__ void load_tile(const float *row, const float *model, uint32_t base, uint32_t n,
                                          float (&a)[4][4])
{
    const uint32_t lane = lane_id();
    if (base + TILE <= n && base + TILE > base) {
        // rows of a server with an odd number of parameters start at odd addresses: 16-byte loads all
        // the same (the hardware asks for 4-byte alignment only)
        f32x4 v[4], m[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = __builtin_nontemporal_load((const f32x4_any *)(row + base + r * 256 + lane * 4));
        if (model) {
#pragma unroll
            for (int r = 0; r < 4; ++r) m[r] = *(const f32x4_any *)(model + base + r * 256 + lane * 4);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) a[r][j] = model ? m[r][j] - v[r][j] : v[r][j];
        return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t e = (uint64_t)base + r * 256 + lane * 4 + j;
            a[r][j] = (e < n) ? (model ? model[e] - row[e] : row[e]) : 0.0f;
        }
}

// The tile's nonzeros in index order through put(position in the tile, element, value); returns how many.
template <class Put>
__device__ __forceinline__ uint32_t each_nonzero(const float (&a)[4][4], uint32_t base, Put put)
{
    const uint32_t lane = lane_id();
    uint32_t run = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        bool f[4];
        uint64_t mk[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f[j] = (__float_as_uint(a[r][j]) & 0x7FFFFFFFu) != 0;
            mk[j] = ballot64(f[j]);
        }
        if ((mk[0] | mk[1] | mk[2] | mk[3]) == 0) continue;
        uint32_t p = run + mbcnt64(mk[0]) + mbcnt64(mk[1]) + mbcnt64(mk[2]) + mbcnt64(mk[3]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (f[j]) put(p++, base + r * 256 + lane * 4 + j, a[r][j]);
        run += (uint32_t)(__popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]));
    }
    return run;
}

__global__ __launch_bounds__(STREAM_THREADS) void k_pull_all_count(const float *row, const float *model, uint32_t n,
                                                                   uint32_t ntiles, uint32_t *tile_cnt, uint2 *slots)
{
    __shared__ uint2 stage_all[WAVES_PER_BLOCK][CAPT];
    const uint32_t wave = uniform(threadIdx.x >> 6), lane = lane_id();
    const uint32_t t = blockIdx.x * WAVES_PER_BLOCK + wave;
    if (t >= ntiles) return;
    float a[4][4];
    load_tile(row, model, t * TILE, n, a);
    uint2 *stage = stage_all[wave];
    const uint32_t cnt = each_nonzero(a, t * TILE, [&](uint32_t p, uint32_t e, float v) {
        if (p < CAPT) stage[p] = make_uint2(e, __float_as_uint(v));
    });
    __builtin_amdgcn_wave_barrier();
    if (cnt <= CAPT) {
        // whole 64-byte lines, as in the streaming pass
        const uint32_t end = (cnt + HEAD - 1u) / HEAD * HEAD;
        for (uint32_t i = lane; i < end; i += 64)
            slots[(size_t)t * CAPT + i] = (i < cnt) ? stage[i] : make_uint2(0u, 0u);
    }
    if (lane == 0) tile_cnt[t] = cnt;
}

// chunk: [0, nc) the chunks' totals, [nc, 2 nc) their first positions.  The total also goes to
// host memory, where the caller reads it once this launch has ended.
__global__ __launch_bounds__(1024) void k_pull_all_scan(const uint32_t *tile_cnt, uint32_t ntiles, uint32_t *tile_pos,
                                                        uint32_t *chunk, uint32_t nc, uint32_t *arrive, uint32_t *total,
                                                        uint32_t *host_total)
{
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t bc;
    constexpr uint32_t PER = PULL_CHUNK / 1024u;
    const uint32_t t0 = blockIdx.x * PULL_CHUNK + threadIdx.x * PER;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        c[i] = (t0 + i < ntiles) ? tile_cnt[t0 + i] : 0u;
        sum += c[i];
    }
    uint32_t tot;
    uint32_t pos = block_excl_scan<16>(sum, wsum, tot);
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        if (t0 + i < ntiles) tile_pos[t0 + i] = pos;
        pos += c[i];
    }
    if (threadIdx.x == 0) st_dev(&chunk[blockIdx.x], tot);
    if (!arrive_last(arrive, nc, &bc)) return;
    uint32_t run = 0;
    for (uint32_t b0 = 0; b0 < nc; b0 += 1024u) {
        const uint32_t b = b0 + threadIdx.x;
        const uint32_t v = (b < nc) ? ld_dev(&chunk[b]) : 0u;
        const uint32_t ex = run + block_excl_scan<16>(v, wsum, tot);
        if (b < nc) chunk[nc + b] = ex;
        run += tot;
    }
    if (threadIdx.x == 0) {
        *total = run;
        __hip_atomic_store(host_total, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// What is sent leaves the row as +0 (D_k -= G), or is added to it (sent_k += G, Eq. 6).
constexpr uint32_t PULL_TPW = 4;      // tiles of one wavefront: their first 64 entries are in flight together

__global__ __launch_bounds__(STREAM_THREADS) void k_pull_all_emit(float *row, const float *model, uint32_t n,
                                                                  uint32_t ntiles, const uint32_t *tile_cnt,
                                                                  const uint32_t *tile_pos, const uint32_t *chunk_base,
                                                                  const uint2 *slots, const uint32_t *total,
                                                                  uint64_t capacity, uint32_t *out_idx, float *out_val)
{
    const uint32_t lane = lane_id();
    const uint32_t t0 = (blockIdx.x * WAVES_PER_BLOCK + uniform(threadIdx.x >> 6)) * PULL_TPW;
    if (*total > capacity) return;
    uint32_t cnt[PULL_TPW], pos[PULL_TPW];
    uint2 first[PULL_TPW];
    float old[PULL_TPW];
#pragma unroll
    for (uint32_t i = 0; i < PULL_TPW; ++i) {
        const uint32_t t = t0 + i;
        cnt[i] = (t < ntiles) ? tile_cnt[t] : 0u;
        pos[i] = (t < ntiles) ? tile_pos[t] + chunk_base[t / PULL_CHUNK] : 0u;
    }
#pragma unroll
    for (uint32_t i = 0; i < PULL_TPW; ++i)
        first[i] = (cnt[i] <= CAPT && lane < cnt[i]) ? slots[(size_t)(t0 + i) * CAPT + lane] : make_uint2(0u, 0u);
    auto put = [&](uint32_t p, uint32_t e, float v, float was) {
        out_idx[p] = e;
        out_val[p] = v;
        store_scattered(&row[e], model ? was + v : 0.0f);
    };
#pragma unroll
    for (uint32_t i = 0; i < PULL_TPW; ++i)
        old[i] = (model && cnt[i] <= CAPT && lane < cnt[i]) ? row[first[i].x] : 0.0f;
#pragma unroll
    for (uint32_t i = 0; i < PULL_TPW; ++i) {
        if (cnt[i] > CAPT) {       // wave-uniform
            float a[4][4];
            load_tile(row, model, (t0 + i) * TILE, n, a);
            each_nonzero(a, (t0 + i) * TILE, [&](uint32_t p, uint32_t e, float v) { put(pos[i] + p, e, v, model ? row[e] : 0.0f); });
            continue;
        }
        if (lane < cnt[i]) put(pos[i] + lane, first[i].x, __uint_as_float(first[i].y), old[i]);
        for (uint32_t q = 64 + lane; q < cnt[i]; q += 64) {
            const uint2 e = slots[(size_t)(t0 + i) * CAPT + q];
            put(pos[i] + q, e.x, __uint_as_float(e.y), model ? row[e.x] : 0.0f);
        }
    }
}

void launch_pull_all(float *row, const float *model, uint32_t n, uint32_t ntiles, uint32_t *tile_cnt, uint2 *slots,
                     uint32_t *scratch, uint32_t *arrive, uint32_t *total, uint32_t *host_total, uint64_t capacity,
                     uint32_t *out_idx, float *out_val, void *stream, void *counted)
{
    hipStream_t st = (hipStream_t)stream;
    const uint32_t nc = (ntiles + PULL_CHUNK - 1) / PULL_CHUNK;
    uint32_t *tile_pos = scratch, *chunk = scratch + ntiles;
    hipLaunchKernelGGL(k_pull_all_count, dim3((ntiles + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK), dim3(STREAM_THREADS), 0,
                       st, row, model, n, ntiles, tile_cnt, slots);
    launch_k(k_pull_all_scan, dim3(nc), dim3(1024), st, nullptr, counted, tile_cnt, ntiles, tile_pos, chunk, nc, arrive,
             total, host_total);
    // (no emission from positions that were not written: the caller reports the error)
    if (hipPeekAtLastError() != hipSuccess || capacity == 0) return;
    constexpr uint32_t per = WAVES_PER_BLOCK * PULL_TPW;
    hipLaunchKernelGGL(k_pull_all_emit, dim3((ntiles + per - 1) / per), dim3(STREAM_THREADS), 0, st, row, model, n,
                       ntiles, tile_cnt, tile_pos, chunk + nc, slots, total, capacity, out_idx, out_val);
}

}  // namespace dgs
