// Internal helpers shared by the libvoxzip kernels and the host API.
// Everything here targets gfx950 (CDNA4): wave64, 160 KB LDS per CU.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/voxzip.h"

namespace vz {

constexpr int kWave = 64;

// ---- bfloat16 <-> float ---------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// Round to nearest, ties to even (finite inputs; NaN becomes a quiet NaN).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu))
        return static_cast<uint16_t>((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

// Element traits: storage type, 16-byte vector width, widening.
template <int DT> struct Elem;
template <> struct Elem<VZ_F32> {
    using T = float;
    static constexpr int kPer16B = 4;
    __device__ static __forceinline__ float load(const T* p, size_t i) { return p[i]; }
    __device__ static __forceinline__ T from_f32(float f) { return f; }
    __device__ static __forceinline__ float to_f32(T x) { return x; }
};
template <> struct Elem<VZ_BF16> {
    using T = uint16_t;
    static constexpr int kPer16B = 8;
    __device__ static __forceinline__ float load(const T* p, size_t i) { return bf16_to_f32(p[i]); }
    __device__ static __forceinline__ T from_f32(float f) { return f32_to_bf16(f); }
    __device__ static __forceinline__ float to_f32(T x) { return bf16_to_f32(x); }
};

// Unpack one 16-byte vector into floats.
template <int DT>
__device__ __forceinline__ void unpack16(const uint4& v, float* out) {
    if constexpr (DT == VZ_F32) {
        out[0] = __uint_as_float(v.x); out[1] = __uint_as_float(v.y);
        out[2] = __uint_as_float(v.z); out[3] = __uint_as_float(v.w);
    } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
}

template <int DT>
__device__ __forceinline__ uint4 pack16(const float* in) {
    uint4 v;
    if constexpr (DT == VZ_F32) {
        v.x = __float_as_uint(in[0]); v.y = __float_as_uint(in[1]);
        v.z = __float_as_uint(in[2]); v.w = __float_as_uint(in[3]);
    } else {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = static_cast<uint32_t>(f32_to_bf16(in[2 * i])) |
                   (static_cast<uint32_t>(f32_to_bf16(in[2 * i + 1])) << 16);
        v.x = w[0]; v.y = w[1]; v.z = w[2]; v.w = w[3];
    }
    return v;
}

// ---- eviction ranking key ---------------------------------------------------
// A larger key is a more important slot: higher score first, then the smaller
// position.  The float is mapped to an order-preserving uint32 (-0 as +0).
__device__ __forceinline__ uint64_t rank_key(float score, int32_t pos) {
    uint32_t b = __float_as_uint(score);
    if (b == 0x80000000u) b = 0u;
    uint32_t ord = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return (static_cast<uint64_t>(ord) << 32) | static_cast<uint64_t>(~static_cast<uint32_t>(pos));
}

// ---- wave / block reductions ------------------------------------------------
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}
// Minimum over the wave (every lane active): the high words first, then the
// low words of the lanes holding that high word; two cross-lane (DPP)
// reductions instead of six dependent 64-bit shuffles through LDS.
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
    const uint32_t hi = static_cast<uint32_t>(v >> 32), lo = static_cast<uint32_t>(v);
    const uint32_t hmin = __reduce_min_sync(~0ull, hi);
    const uint32_t lmin = __reduce_min_sync(~0ull, hi == hmin ? lo : 0xFFFFFFFFu);
    return (static_cast<uint64_t>(hmin) << 32) | lmin;
}
// Max and sum over the 16 lanes of a DPP row, in every lane (rotations by 8,
// 4, 2 and 1; each step combines the same two values in both lanes of a pair).
template <int ROR>
__device__ __forceinline__ float ror16(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + ROR, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, ror16<8>(v));
    v = fmaxf(v, ror16<4>(v));
    v = fmaxf(v, ror16<2>(v));
    return fmaxf(v, ror16<1>(v));
}
__device__ __forceinline__ float row16_sum(float v) {
    v += ror16<8>(v);
    v += ror16<4>(v);
    v += ror16<2>(v);
    return v + ror16<1>(v);
}
// The same across the wave's four rows (lanes l, l ^ 16, l ^ 32, l ^ 48): row
// swaps in registers, with the values and order of shuffles by 16 and then 32.
__device__ __forceinline__ float rows_max(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// ---- softmax statistics of a head from its chunks' pairs ----
// (max and sum of exp of each chunk, from ml on), by the 16 lanes of a DPP row: lane i takes chunks i,
// i + 16, ....  Every lane of the row gets the sequence's pair.  Up to
// kPairChunks chunks: at most eight pairs per lane, all loaded (indexes
// clamped) before any is used, in rounds of 16 chunks of which those past
// n_load are left out (uniform); merge_all takes any number, with the same
// order of additions.  rel(x, m): exp of x relative to m, 0 for x = -inf.
constexpr int kPairs = 8;
constexpr int kPairChunks = 16 * kPairs;
__device__ __forceinline__ void load_pairs(const float2* ml, int n_load, int c0, float2 (&p)[kPairs]) {
#pragma unroll
    for (int k = 0; k < kPairs; ++k) {
        p[k] = make_float2(-INFINITY, 0.f);
        if (16 * k < n_load) p[k] = ml[min(c0 + 16 * k, n_load - 1)];
    }
}
template <class Rel>
__device__ __forceinline__ float2 merge_pairs(const float2 (&p)[kPairs], int nc, int i, Rel rel) {
    float m = -INFINITY, z = 0.f;
#pragma unroll
    for (int k = 0; k < kPairs; ++k) m = fmaxf(m, i + 16 * k < nc ? p[k].x : -INFINITY);
    m = row16_max(m);
#pragma unroll
    for (int k = 0; k < kPairs; ++k) {
        if (16 * k >= nc) break;
        const float f = rel(i + 16 * k < nc ? p[k].x : -INFINITY, m);
        z = fmaf(i + 16 * k < nc ? p[k].y : 0.f, f, z);
    }
    return make_float2(m, row16_sum(z));
}
// The sum of a head's pairs relative to their max m.
template <class Rel>
__device__ __forceinline__ float merge_sum(const float2* ml, int nc, int i, float m, Rel rel) {
    float2 p[kPairs];
    float z = 0.f;
    for (int c0 = i; c0 - i < nc; c0 += kPairChunks) {
        load_pairs(ml, nc, c0, p);
#pragma unroll
        for (int k = 0; k < kPairs; ++k) {
            const float f = rel(c0 + 16 * k < nc ? p[k].x : -INFINITY, m);
            z = fmaf(c0 + 16 * k < nc ? p[k].y : 0.f, f, z);
        }
    }
    return row16_sum(z);
}
template <class Rel>
__device__ __forceinline__ float2 merge_all(const float2* ml, int nc, int i, Rel rel) {
    float2 p[kPairs];
    float m = -INFINITY;
    for (int c0 = i; c0 - i < nc; c0 += kPairChunks) {
        load_pairs(ml, nc, c0, p);
#pragma unroll
        for (int k = 0; k < kPairs; ++k) m = fmaxf(m, p[k].x);  // a clamped pair is one of the head's own
    }
    m = row16_max(m);
    return make_float2(m, merge_sum(ml, nc, i, m, rel));
}

// Inclusive wave scan (DPP row shifts, then the row totals broadcast upwards).
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ int wave_sum_i(int v) { return __builtin_amdgcn_readlane(wave_incl_scan(v), kWave - 1); }

}  // namespace vz

// ---- ragged batches ---------------------------------------------------------
// Sequence s of a ragged batch owns slots base[s] .. base[s] + cap[s] - 1 of
// every (layer, head) plane, and a plane holds `total` slots.  The
// per-sequence values are device arrays read by the kernels; a sequence whose
// values are out of range is skipped (nothing of it is read or written) and
// its status entry says why.
struct VzRagged {
    const int64_t* base;
    const int32_t* cap;
    const int32_t* len;
    const int32_t* next_pos;
    const int32_t* budget;  // eviction only
    int32_t* status;        // [n], may be null
    int32_t n;
    int64_t total;
};

// Largest plane (slots) and batch a ragged call serves: every flat chunk index
// and running count below stays far from 2^31.
constexpr int64_t kRaggedMaxTotal = int64_t(1) << 26;
constexpr int32_t kRaggedMaxSeqs = 1 << 15;  // also a grid dimension

namespace vz {

// Status of a sequence for a decode step from its values (base, cap, len,
// next_pos): VZ_OK when slot len exists and the sequence lies inside the
// planes of `total` slots, VZ_IDLE for an idle slot (cap 0).
__device__ __forceinline__ int decode_status_of(int64_t b, int c, int n, int p, int64_t total) {
    if (c == 0) return VZ_IDLE;
    if (n < 0 || p < 0 || c < 1 || b < 0 || b > total - c) return VZ_ERR_INVALID;
    if (n >= c) return VZ_ERR_CAPACITY;  // no free slot (len + 1 > cap, without overflow)
    return VZ_OK;
}
// decode_status_of(...) == VZ_OK without branches: a value loaded for it is
// not loaded behind the check of another.
__device__ __forceinline__ bool decode_served(int64_t b, int c, int n, int p, int64_t total) {
    return (c > 0) & (n >= 0) & (p >= 0) & (b >= 0) & (b <= total - c) & (n < c);
}
__device__ __forceinline__ int ragged_decode_status(const VzRagged& r, int s) {
    return decode_status_of(r.base[s], r.cap[s], r.len[s], r.next_pos[s], r.total);
}

// Keys are handled in chunks of kChunk by the decode paths that keep per-chunk
// results in the workspace.
constexpr int kChunk = 128;

// Chunks of sequence s in a ragged call (0 when it cannot be served).
__device__ __forceinline__ int ragged_chunks(const VzRagged& r, int s) {
    const int n = r.len[s];
    return decode_served(r.base[s], r.cap[s], n, r.next_pos[s], r.total) ? (n + kChunk) / kChunk : 0;
}

// The sequence a work item belongs to, resolved at the top of every kernel.
struct SeqItem {
    int s;           // sequence (0 for a single-sequence call)
    int len, next_pos;
    int n_chunks;    // chunks of the sequence
    int first;       // its first chunk row in the workspace
    int64_t base;    // its first slot in the planes
};

// Flat chunk f of a ragged call, found by a whole wave: each lane loads one
// sequence's values (64 sequences per round), a wave scan of their chunk
// counts finds the owner of f, and the owner's values are taken from the lane
// that loaded them, so the kernel waits for one round of loads.  A call of one
// sequence needs no search (scalar loads only).  False when f lies past the
// call's chunks (or past the nc_max rows).
__device__ __forceinline__ bool locate_ragged_chunk(const VzRagged& r, int nc_max, int f, SeqItem& it, int& c) {
    if (r.n == 1) {
        it.s = 0;
        it.base = r.base[0];
        it.len = r.len[0];
        it.next_pos = r.next_pos[0];
        const bool ok = decode_served(it.base, r.cap[0], it.len, it.next_pos, r.total);
        it.n_chunks = (it.len + kChunk) / kChunk;
        it.first = 0;
        c = f;
        return ok && f < it.n_chunks && it.n_chunks <= nc_max;
    }
    const int lane = threadIdx.x % kWave;
    int run = 0;
    for (int s0 = 0; s0 < r.n && run <= nc_max; s0 += kWave) {
        const int su = min(s0 + lane, r.n - 1);  // load for every lane, mask after
        const int64_t b = r.base[su];
        const int cp = r.cap[su], ln = r.len[su], np = r.next_pos[su];
        const bool ok = (s0 + lane < r.n) & decode_served(b, cp, ln, np, r.total);
        const int n = ok ? (ln + kChunk) / kChunk : 0;
        const int incl = wave_incl_scan(n);
        const unsigned long long hit = __ballot(run + incl > f);
        if (hit) {
            const int src = __builtin_ctzll(hit);
            const int nc = __builtin_amdgcn_readlane(n, src);
            const int first = run + __builtin_amdgcn_readlane(incl, src) - nc;
            if (first + nc > nc_max) return false;
            it.s = s0 + src;
            it.len = __builtin_amdgcn_readlane(ln, src);
            it.next_pos = __builtin_amdgcn_readlane(np, src);
            const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(b), src);
            const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), src);
            it.base = static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
            it.n_chunks = nc;
            it.first = first;
            c = f - first;
            return true;
        }
        run += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    return false;
}

// First flat item of sequence t when sequence s contributes count(s) >= 0
// consecutive items, in sequence order, or -1 when it lies past `limit`.
// Called by a whole wave (every lane gets the same result).
template <class Count>
__device__ int ragged_first(int t, int limit, Count count) {
    const int lane = threadIdx.x % kWave;
    int run = 0;
    for (int s0 = 0; s0 < t && run <= limit; s0 += kWave) {
        const int s = s0 + lane;
        const int n0 = count(s < t ? s : t - 1);
        run += wave_sum_i(s < t ? n0 : 0);
    }
    return run <= limit ? __builtin_amdgcn_readfirstlane(run) : -1;
}

}  // namespace vz

// ---- launchers (one per kernel family), called by the host API -------------
struct VzDecodeArgs {
    const void* q; const void* k_new; const void* v_new;
    void* k_cache; void* v_cache; float* score; int32_t* pos; void* out;
    int32_t len, next_pos; float gamma, sm_scale;
    int32_t L, Hq, Hkv, d, cap, dtype;
    void* ws; size_t ws_bytes;
    // ragged batch (rag.n > 0): len, next_pos and cap above are unused; q, out
    // are [n][L][Hq][d], k_new, v_new [n][L][Hkv][d], planes hold rag.total slots
    VzRagged rag;
    // a single sequence for which vz_decode_evicts says so: the eviction of
    // the len + 1 slots the step leaves runs in the decode launches (ev = 1), with these arguments; ev_n is the
    // eviction workspace's move-count array
    int32_t ev, ev_budget, ev_sink, ev_M;
    int32_t* ev_kept;
    int32_t* ev_n;
};

struct VzEvictArgs {
    void* k_cache; void* v_cache; float* score; int32_t* pos;
    int32_t len, budget, n_sink, n_recent, next_pos;
    int32_t* kept_pos_out;
    int32_t L, Hkv, d, cap, dtype;
    void* ws; size_t ws_bytes;
    // ragged batch (rag.n > 0): len, budget, next_pos and cap above are unused;
    // kept_pos_out is [L][rag.total] (sequence s from slot base[s]); new_len_out
    // receives min(len, budget) per sequence
    VzRagged rag;
    int32_t* new_len_out;
};

// Stage-1 span offsets (host); arguments checked by the caller; returns the
// number of spans written to off_out[1..].
int32_t vz_build_span_offsets(const int64_t* t_start_ms, const int64_t* t_end_ms, const float* conf,
                              const int32_t* text_len, int32_t n_seg, int64_t t_total_ms, int32_t L_a,
                              float conf_threshold, int32_t* off_out);
hipError_t vz_launch_fuse(const void* k_in, const void* v_in, int32_t T_in, const int32_t* off,
                          int32_t n_spans, const void* ak, const void* av, void* k_out, void* v_out,
                          float* score_out, int32_t* pos_out, int32_t L, int32_t H, int32_t d,
                          int32_t cap_out, int32_t dtype, hipStream_t stream);
struct VzFuseRaggedArgs {
    const void* k_in; const void* v_in;
    const int64_t* in_base; const int32_t* T_in;
    const int32_t* span_off; const int64_t* off_base; const int32_t* n_spans;
    const void* anchor_k; const void* anchor_v;
    void* k_out; void* v_out; float* score_out; int32_t* pos_out;
    const int64_t* seq_base; const int32_t* cap; int32_t* status;
    int32_t n_seqs; int64_t total_in, total_off, total; int32_t max_spans;
    int32_t L, Hkv, d, dtype;
};
hipError_t vz_launch_fuse_ragged(const VzFuseRaggedArgs& a, hipStream_t stream);
// Decode sizing: plane = slots per (layer, KV head) plane (cap, or the total
// of a ragged batch); n_seqs = 0 for a single sequence.
size_t vz_decode_ws_bytes(int32_t L, int32_t Hq, int32_t Hkv, int32_t d, int64_t plane, int32_t n_seqs);
// decode workspace: a header of vz_decode_hdr_bytes(L) bytes, then
// path-specific scratch
size_t vz_decode_hdr_bytes(int32_t L);
bool vz_decode_fused_ok(int32_t dtype, int32_t d, int32_t Hq, int32_t Hkv, int32_t L, int64_t plane, int32_t n_seqs);
// Workspace of the chunked path and of the general path (the same layout of
// rows: per (layer, chunk row, query head) one float2 and 512 bytes).
size_t vz_decode_fused_ws_bytes(int32_t L, int32_t Hq, int64_t plane, int32_t n_seqs);
// Chunk rows per layer of either path's workspace.
int64_t vz_decode_chunk_rows(int64_t plane, int32_t n_seqs);
hipError_t vz_launch_decode_fused(const VzDecodeArgs& a, hipStream_t stream);
hipError_t vz_launch_decode_generic(const VzDecodeArgs& a, hipStream_t stream);
hipError_t vz_launch_decode(const VzDecodeArgs& a, hipStream_t stream);
// Whole-range decode path (single sequence): whether a call takes it.
bool vz_decode_takes_range(const VzDecodeArgs& a);
// Workspace of the whole-range path (single sequence or ragged batch).
size_t vz_decode_range_ws_bytes(int32_t L, int32_t Hq, int32_t Hkv, int64_t plane, int32_t n_seqs);
// Whether a decode call's launches also run the eviction of the len + 1 slots
// it leaves: on the whole-range path in one part with Hkv <= 4 and at most 256
// moved rows; on the other paths one eviction (T = budget + 1) with no kept
// positions asked for.
bool vz_decode_evicts(const VzDecodeArgs& a, int32_t budget, bool kept);
// The layers' arrival counters of a decode workspace's header (whole-range
// path).
uint64_t* vz_decode_counters(void* ws);
// A fresh nonzero tag per call (arrival counters of the whole-range path).
uint32_t vz_call_tag();
size_t vz_evict_ws_bytes(int32_t L, int64_t plane, int32_t n_seqs);
hipError_t vz_launch_evict(const VzEvictArgs& a, hipStream_t stream);
