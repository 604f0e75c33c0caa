// Decode step (Sec. 3.1 Eq. 1-2, Sec. 3.2.2 Eq. 6), general path: any group
// size up to 16, float32 or bfloat16, d in {64, 128}.  It serves float32
// caches, head size 64 and the head groups that the bfloat16 d = 128 paths do
// not take.  Logits, probabilities and every sum are float32 in both element
// types; keys are handled in chunks of 128 as on the chunked path.
//
//   logits   one workgroup per (layer, KV head, chunk), four waves of 32 keys:
//            S^T = K Q^T on the matrix cores (16 keys x 16 query heads), the
//            logits to the workspace, the chunk's max and sum of exp per head;
//            the workgroup whose chunk holds slot len appends the new row
//            first and reads it from k_new;
//   values   one workgroup per (layer, KV head, run of chunks): the sequence's
//            softmax statistics from the chunks' pairs, p from the logits,
//            O^T = V^T P^T on the matrix cores and each key's sum over the
//            group's heads of p, which takes the place of the logits it was
//            formed from; so does the run's output when there are several;
//   finish   Eq. (6) from the key sums of the KV heads, and the output rows
//            from the runs' outputs (not launched when the values kernel has
//            done both: one KV head and one run).
//
// Both products stream their rows straight from the cache into the MFMA
// operand layouts, with no trip through LDS: float32 rows (and float32 p) take
// v_mfma_f32_16x16x4_f32, bfloat16 keys v_mfma_f32_16x16x32_bf16 (products of
// bfloat16 are exact in float32); bfloat16 values are widened first, so that p
// keeps its 24 bits.  At 16 heads the float32 instruction needs about a
// quarter of its rate to keep up with HBM, so large calls are bound by memory
// and small ones by the launches and the round trips inside each.  Measured,
// whole passes (before: one thread per key for the logits, one workgroup per
// (layer, head) for softmax and P V, one thread per key for the scores):
//   16 layers, 16Q/4KV, d = 128, float32, 2049 keys, with the eviction
//                                                     499 -> 44.4 us (3.0 TB/s)
//   24 layers, 14Q/2KV, d = 64, bfloat16, 4001 keys   343 -> 22.0 us (2.2 TB/s)
//   1 layer, 4Q/1KV, d = 64, float32, 129 keys, with the eviction
//                                                     26.7 -> 14.4 us, of which 10.6 kernels
#include <math.h>

#include <type_traits>

#include "select.h"

namespace {

using vz::SeqItem;
using vz::kChunk;
using vz_sel::kBufferDword3;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / vz::kWave;
constexpr int kKeysPerWave = kChunk / kWaves;  // 32: two 16-key tiles
constexpr int kHeads = 16;                     // head columns of a matrix instruction, and the largest group
constexpr int kMaxRuns = 64;                   // runs of chunks per sequence
constexpr int kStatChunks = vz::kPairChunks;   // chunks whose pairs the values kernel merges itself

// Arguments of the launches (a single-sequence call has rag.n == 0).
struct GenericArgs {
    const void* q;
    const void* k_new;
    const void* v_new;
    void* k_cache;
    void* v_cache;
    int32_t* pos;
    float* score;
    void* out;
    float* S;        // logits [L][nc_max][Hq][kChunk], then key sums and run outputs in their place
    float2* ml;      // max and sum of exp per (layer, head, chunk row) [L][Hq][nc_max]
    float2* layer;   // the same per (sequence, layer, head), for planes of more than kStatChunks chunks (else free)
    int32_t len, next_pos, n_chunks;  // single sequence
    int32_t nc_max;                   // chunk rows per layer
    int32_t Hq, Hkv, L;
    int64_t plane;
    float scale, gamma;
    VzRagged rag;
    vz_sel::EvictOne ev;              // a single sequence's eviction, by the launch that folds
};

// The same search as vz::locate_ragged_chunk for batches of more than kManySeqs
// sequences: kSeqRounds rounds of 64 sequences loaded at once.  With a block
// per chunk and KV head, the rounds' load latencies one after another are most
// of such a call's time when its sequences are short (16 heads and KV heads,
// 2,000 sequences of 20 keys: one layer 856 -> 695 us, 8 layers 6,820 -> 5,430;
// 14 / 2 heads, d = 64: one layer 177 -> 165, but 513 of 20 keys 30.1 -> 31.7 and
// 8 layers, 300 of 10-1,500 keys 428 -> 448: not used there).
constexpr int kManySeqs = 1024, kSeqRounds = 8;
__device__ __forceinline__ bool locate_chunk_of_many(const VzRagged& r, int nc_max, int f, SeqItem& it, int& c) {
    const int lane = threadIdx.x % vz::kWave;
    int run = 0;
    for (int s0 = 0; s0 < r.n; s0 += kSeqRounds * vz::kWave) {
        int64_t b[kSeqRounds];
        int cp[kSeqRounds], ln[kSeqRounds], np[kSeqRounds];
#pragma unroll
        for (int k = 0; k < kSeqRounds; ++k) {
            const int su = min(s0 + k * vz::kWave + lane, r.n - 1);  // load for every lane, mask after
            b[k] = r.base[su];
            cp[k] = r.cap[su];
            ln[k] = r.len[su];
            np[k] = r.next_pos[su];
        }
#pragma unroll
        for (int k = 0; k < kSeqRounds; ++k) {
            const bool ok = (s0 + k * vz::kWave + lane < r.n) & vz::decode_served(b[k], cp[k], ln[k], np[k], r.total);
            const int n = ok ? (ln[k] + kChunk) / kChunk : 0;
            const int incl = vz::wave_incl_scan(n);
            const unsigned long long hit = __ballot(run + incl > f);
            if (hit) {
                const int src = __builtin_ctzll(hit);
                it.n_chunks = __builtin_amdgcn_readlane(n, src);
                it.first = run + __builtin_amdgcn_readlane(incl, src) - it.n_chunks;
                it.s = s0 + k * vz::kWave + src;
                it.len = __builtin_amdgcn_readlane(ln[k], src);
                it.next_pos = __builtin_amdgcn_readlane(np[k], src);
                const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(b[k]), src);
                const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(b[k] >> 32), src);
                it.base = static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
                c = f - it.first;
                return it.first + it.n_chunks <= nc_max;
            }
            run += __builtin_amdgcn_readlane(incl, vz::kWave - 1);
            if (run > nc_max) return false;
        }
    }
    return false;
}

// Flat chunk f of a layer: false when it holds no work; c = chunk inside the
// sequence.  RAG: 0 a single sequence, 1 a ragged batch, 2 one of many
// sequences.
template <int RAG>
__device__ __forceinline__ bool resolve_chunk(const GenericArgs& a, int f, SeqItem& it, int& c) {
    if constexpr (RAG == 2) {
        return locate_chunk_of_many(a.rag, a.nc_max, f, it, c);
    } else if constexpr (RAG == 1) {
        return vz::locate_ragged_chunk(a.rag, a.nc_max, f, it, c);
    } else {
        it = SeqItem{0, a.len, a.next_pos, a.n_chunks, 0, 0};
        c = f;
        return f < a.n_chunks;
    }
}

// Runs of a sequence of nc chunks: runs of `step` chunks, the last one taking
// the remainder as well.  A run's output replaces logits of the run's first
// two chunks, so runs have at least two chunks; with one head per KV head
// there is no room beside the key sums, and a sequence is one run.
// (Function of the sequence and the group size alone: a ragged call gives the
// bits of a single-sequence call.)
struct Runs {
    int n, step;
};
__host__ __device__ inline Runs runs_of(int nc, int G) {
    Runs r;
    r.step = max(2, (nc + kMaxRuns - 1) / kMaxRuns);
    r.n = G == 1 ? 1 : max(1, nc / r.step);
    return r;
}

// Row (layer, chunk row, head) of the logits; a head's pairs.
__device__ __forceinline__ size_t ws_row(const GenericArgs& a, int l, int chunk_row, int h) {
    return (static_cast<size_t>(l) * a.nc_max + chunk_row) * a.Hq + h;
}
__device__ __forceinline__ float2* ml_of(const GenericArgs& a, int l, int h) {
    return a.ml + (static_cast<size_t>(l) * a.Hq + h) * a.nc_max;
}
// Run output of head hg of KV head g (first chunk row `row` of the run): heads
// 1 .. in their own rows of that chunk, head 0 in row 1 of the next one (rows
// 0 hold the key sums).
__device__ __forceinline__ float* run_out(const GenericArgs& a, int l, int row, int g, int G, int hg) {
    return a.S + (hg > 0 ? ws_row(a, l, row, g * G + hg) : ws_row(a, l, row + 1, g * G + 1)) * kChunk;
}

// exp(x - m), 0 for an absent x (-inf, also when m is -inf).
__device__ __forceinline__ float exp_rel(float x, float m) { return x == -INFINITY ? 0.f : expf(x - m); }

// PACK: groups of at most 8 heads, whose second tile's logits are rotated into
// head columns 8..15, so every exp serves a key and a head that exist.
template <int DT, int D, int RAG, bool PACK>
__global__ __launch_bounds__(kThreads) void logits_kernel(const GenericArgs a) {
    using E = vz::Elem<DT>;
    using T = typename E::T;
    constexpr int PER = E::kPer16B;
    constexpr int NV = D / (4 * PER);  // 16-byte pieces of a row per lane: channels 4 PER s + PER q4 ..
    constexpr int NS = PACK ? 1 : 2;   // sets of four logits per lane
    __shared__ float s_m[kWaves][kHeads], s_l[kWaves][kHeads];
    const int l = blockIdx.y, g = blockIdx.z;
    SeqItem it;
    int c;
    if (!resolve_chunk<RAG>(a, blockIdx.x, it, c)) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / vz::kWave), lane = tid % vz::kWave;
    const int q4 = lane >> 4, r16 = lane & 15;
    const int Hq = a.Hq, G = Hq / a.Hkv, len = it.len;
    const size_t row_sl = static_cast<size_t>(it.s) * a.L + l;
    const size_t head = (static_cast<size_t>(l) * a.Hkv + g) * a.plane + it.base;
    T* const K = static_cast<T*>(a.k_cache) + head * D;
    T* const V = static_cast<T*>(a.v_cache) + head * D;
    const T* const kn = static_cast<const T*>(a.k_new) + (row_sl * a.Hkv + g) * D;
    const T* const vn = static_cast<const T*>(a.v_new) + (row_sl * a.Hkv + g) * D;

    // rows of the wave's two tiles (past the new one: the new row again, masked)
    const int k0 = c * kChunk + kKeysPerWave * w;
    uint4 kr[2][NV], qr[NV];
    if (k0 + kKeysPerWave <= len) {  // wave-uniform: all in the cache, one address and immediate offsets
        const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(K + static_cast<size_t>(k0) * D, 0,
                                                                            kKeysPerWave * D * sizeof(T), kBufferDword3);
        const int off = (r16 * D + PER * q4) * static_cast<int>(sizeof(T));
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int s = 0; s < NV; ++s)
                kr[ti][s] = __builtin_bit_cast(
                    uint4, __builtin_amdgcn_raw_buffer_load_b128(rk, off + 64 * s, ti * 16 * D * sizeof(T), 0));
    } else {
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
            const int key = k0 + 16 * ti + r16;
            const T* row = key < len ? K + static_cast<size_t>(key) * D : kn;
#pragma unroll
            for (int s = 0; s < NV; ++s) kr[ti][s] = *reinterpret_cast<const uint4*>(row + PER * (4 * s + q4));
        }
    }
    {
        const T* row = static_cast<const T*>(a.q) + (row_sl * Hq + g * G + min(r16, G - 1)) * D;
#pragma unroll
        for (int s = 0; s < NV; ++s) __builtin_memcpy(&qr[s], row + PER * (4 * s + q4), 16);  // any element alignment
    }
    // Eq. (1): the new row, after this workgroup's loads of the chunk
    if (c == len / kChunk) {
        constexpr int CH = D / PER;
        if (tid < 2 * CH) {
            const int o = PER * (tid % CH);
            T* dst = (tid < CH ? K : V) + static_cast<size_t>(len) * D + o;
            *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>((tid < CH ? kn : vn) + o);
        }
        if (!RAG && a.ev.cnt && g == 0 && tid == 2 * CH) a.ev.cnt[l * static_cast<size_t>(a.ev.stride)] = 0;  // counted by the launch that folds
        if (g == 0 && tid == 2 * CH) a.pos[static_cast<size_t>(l) * a.plane + it.base + len] = it.next_pos;
    }
    if (r16 >= G) {  // unused head columns
#pragma unroll
        for (int s = 0; s < NV; ++s) qr[s] = make_uint4(0, 0, 0, 0);
    }
    f32x4 acc[2];
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
        acc[ti] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NV; ++s) {
            if constexpr (DT == VZ_F32) {
                const float kf[4] = {__uint_as_float(kr[ti][s].x), __uint_as_float(kr[ti][s].y),
                                     __uint_as_float(kr[ti][s].z), __uint_as_float(kr[ti][s].w)};
                const float qf[4] = {__uint_as_float(qr[s].x), __uint_as_float(qr[s].y), __uint_as_float(qr[s].z),
                                     __uint_as_float(qr[s].w)};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[ti] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i], qf[i], acc[ti], 0, 0, 0);
            } else {
                bf16x8_t kf, qf;
                __builtin_memcpy(&kf, &kr[ti][s], 16);
                __builtin_memcpy(&qf, &qr[s], 16);
                acc[ti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf, acc[ti], 0, 0, 0);
            }
        }
    }
    // lane: head hc, keys 16 (ti or half) + 4 q4 + i
    const int hc = PACK ? r16 & 7 : r16, half = PACK ? r16 >> 3 : 0;
    float* const S = a.S + ws_row(a, l, it.first + c, g * G + hc) * kChunk + kKeysPerWave * w + 16 * half + 4 * q4;
    float sv[NS][4], m_w = -INFINITY;
#pragma unroll
    for (int ti = 0; ti < NS; ++ti) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x = acc[ti][i];
            if constexpr (PACK) {
                const float second = vz::ror16<8>(acc[1][i]);
                x = half ? second : x;
            }
            sv[ti][i] = k0 + 16 * (ti + half) + 4 * q4 + i <= len ? x * a.scale : -INFINITY;
            m_w = fmaxf(m_w, sv[ti][i]);
        }
        if (hc < G)
            *reinterpret_cast<float4*>(S + 16 * ti) = make_float4(sv[ti][0], sv[ti][1], sv[ti][2], sv[ti][3]);
    }
    m_w = vz::rows_max(m_w);
    if constexpr (PACK) m_w = fmaxf(m_w, vz::ror16<8>(m_w));
    float l_w = 0.f;
#pragma unroll
    for (int ti = 0; ti < NS; ++ti)
#pragma unroll
        for (int i = 0; i < 4; ++i) l_w += exp_rel(sv[ti][i], m_w);
    l_w = vz::rows_sum(l_w);
    if constexpr (PACK) l_w += vz::ror16<8>(l_w);
    if (q4 == 0) {
        s_m[w][r16] = m_w;
        s_l[w][r16] = l_w;
    }
    __syncthreads();
    if (tid < G) {
        float m = s_m[0][tid], z = 0.f;
#pragma unroll
        for (int v = 1; v < kWaves; ++v) m = fmaxf(m, s_m[v][tid]);
#pragma unroll
        for (int v = 0; v < kWaves; ++v) z = fmaf(s_l[v][tid], exp_rel(s_m[v][tid], m), z);
        ml_of(a, l, g * G + tid)[it.first + c] = make_float2(m, z);
    }
}

struct ExpRel {
    __device__ __forceinline__ float operator()(float x, float m) const { return exp_rel(x, m); }
};

// Statistics of every head of a (sequence, layer), once, for calls whose
// planes hold more than kStatChunks chunks (where merging them in every
// workgroup of the values kernel would read chunks x runs pairs).
template <bool RAG>
__global__ __launch_bounds__(kThreads) void stats_kernel(const GenericArgs a) {
    const int l = blockIdx.y, s = blockIdx.z;
    int first = 0, nc = a.n_chunks;
    if constexpr (RAG) {
        nc = vz::ragged_chunks(a.rag, s);
        first = vz::ragged_first(s, a.nc_max, [&](int u) { return vz::ragged_chunks(a.rag, u); });
        if (nc == 0 || first < 0 || first + nc > a.nc_max) return;
    }
    const int h = blockIdx.x * (kThreads / 16) + threadIdx.x / 16, i = threadIdx.x % 16;
    const float2 st = vz::merge_all(ml_of(a, l, min(h, a.Hq - 1)) + first, nc, i, ExpRel());
    if (i == 0 && h < a.Hq) a.layer[(static_cast<size_t>(s) * a.L + l) * a.Hq + h] = st;
}

// Sums over the lanes of a DPP row that hold a key's heads, in every lane: all
// 16, or (PACK) the 8 of each half row.
template <bool PACK>
__device__ __forceinline__ float heads_sum(float v) {
    if constexpr (!PACK) return vz::row16_sum(v);
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});         // quad_perm [1, 0, 3, 2]
    v += dpp(v, std::integral_constant<int, 0x4E>{});         // quad_perm [2, 3, 0, 1]
    return v + dpp(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
}

// Values of a row piece (four or eight channels of one key) as floats.
template <int DT, int PER>
__device__ __forceinline__ void widen(const uint32_t* x, float* f) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if constexpr (DT == VZ_F32) f[i] = __uint_as_float(x[i]);
        else f[i] = __uint_as_float((i & 1) ? x[i / 2] & 0xFFFF0000u : x[i / 2] << 16);
    }
}

// The eviction of a layer, by the block that folded its last scores.
template <int NT, class T, int D>
__device__ void evict_layer(const GenericArgs& a, int l) {
    const size_t row = static_cast<size_t>(l) * a.plane;
    vz_sel::evict_one_slot<NT, T, D>(a.ev, a.score + row, a.pos + row, static_cast<T*>(a.k_cache) + row * a.Hkv * D,
                                     static_cast<T*>(a.v_cache) + row * a.Hkv * D, static_cast<size_t>(a.plane) * D,
                                     a.Hkv, a.len + 1, a.next_pos + 1);
}

// PACK (groups of at most 8 heads): lanes r16 >= 8 of a row hold the heads of
// the second 16 keys of a wave's 32, so every exp serves a key and a head that
// exist; a rotation by 8 lanes makes them the second tile's B operand (the
// other columns of either product hold heads that are not read).
template <int DT, int D, int RAG, bool PACK>
__global__ __launch_bounds__(kThreads) void values_kernel(const GenericArgs a) {
    using E = vz::Elem<DT>;
    using T = typename E::T;
    // Lane (q4, r16) loads channels PER r16 .. + PER - 1 (of each of NP
    // pieces of a row) of keys 4 q4 + i: component e of piece j is row r16 of
    // the A operand of output tile PER j + e, key 4 q4 + i its column q4.
    constexpr int PER = DT == VZ_F32 ? 4 : D / 16;
    constexpr int NP = D / (16 * PER);
    constexpr int NT = D / 16;                          // output tiles
    constexpr int WORDS = PER * sizeof(T) / 4;
    constexpr int DEPTH = NP * WORDS <= 2 ? 2 : 1;      // 32-key units in flight per wave (16, 32 or 64 registers each)
    constexpr int NS = PACK ? 1 : 2;                    // logit pieces of a unit per lane
    __shared__ float s_o[kWaves][kHeads][D + 4];
    __shared__ float2 s_stat[kHeads];
    const int l = blockIdx.y, g = blockIdx.z;
    const int Hq = a.Hq, G = Hq / a.Hkv;
    SeqItem it;
    int c0, run;
    Runs rn;
    if constexpr (RAG) {
        // grid over chunk rows: the first chunk of each run works
        if (!resolve_chunk<RAG>(a, blockIdx.x, it, c0)) return;
        rn = runs_of(it.n_chunks, G);
        run = c0 / rn.step;
        if (run >= rn.n || c0 != run * rn.step) return;
    } else {
        resolve_chunk<0>(a, 0, it, c0);
        rn = runs_of(it.n_chunks, G);
        run = blockIdx.x;
        c0 = run * rn.step;
    }
    const int nch = (run == rn.n - 1 ? it.n_chunks : c0 + rn.step) - c0;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / vz::kWave), lane = tid % vz::kWave;
    const int q4 = lane >> 4, r16 = lane & 15;
    const int hc = PACK ? r16 & 7 : r16, half = PACK ? r16 >> 3 : 0;  // the lane's head, and 16 keys of a unit
    const int len = it.len;
    const size_t row_sl = static_cast<size_t>(it.s) * a.L + l;
    const T* const V =
        static_cast<const T*>(a.v_cache) + ((static_cast<size_t>(l) * a.Hkv + g) * a.plane + it.base) * D;
    float* const sc = a.score + static_cast<size_t>(l) * a.plane + it.base;
    const bool fold = a.Hkv == 1;  // one KV head: its key sums are the whole of Eq. (6)'s

    // Unit x of the wave: keys 32 w .. + 31 of chunk c0 + x, two tiles of 16.
    // Scalar descriptors bound every access, so an address is one lane offset
    // and an immediate: heads past the group and rows past the new one read
    // as zero (their p is 0: the logits of keys past the new one are -inf, the
    // max of heads past the group +inf).
    auto unit_key = [&](int x) { return (c0 + x) * kChunk + kKeysPerWave * w; };
    auto logits_of = [&](int x) {
        return __builtin_amdgcn_make_buffer_rsrc(
            a.S + ws_row(a, l, it.first + c0 + x, g * G) * kChunk, 0,
            __builtin_amdgcn_readfirstlane(G * kChunk * 4), kBufferDword3);
    };
    // a plane's `bytes` per key, for `keys` keys from k0 on of those below n
    auto keys_of = [&](const void* p, int k0, int n, int bytes, int keys) {
        return __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(static_cast<const char*>(p)) + static_cast<size_t>(k0) * bytes, 0,
            __builtin_amdgcn_readfirstlane(min(max(n - k0, 0), keys) * bytes), kBufferDword3);
    };
    const int s_off = 4 * (hc * kChunk + kKeysPerWave * w + 16 * half + 4 * q4);
    struct Logits {
        float4 s;
        float old;  // when this kernel folds: the old score of the key the lane will store (0 for the new slot)
    };
    const int key_off = 16 * half + 4 * q4 + (r16 & 3);  // the lane's key of the 16 or 32 it sums for
    auto load_s = [&](int x, Logits (&p)[NS]) {
        const __amdgpu_buffer_rsrc_t rs = logits_of(x);
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            p[h].s = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, s_off + 64 * h, 0, 0));
            if (fold) {
                const __amdgpu_buffer_rsrc_t ro = keys_of(sc, unit_key(x) + 16 * h, len, 4, PACK ? 32 : 16);
                p[h].old = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ro, 4 * key_off, 0, 0));
            }
        }
    };
    const int v_off = (4 * q4 * D + PER * r16) * static_cast<int>(sizeof(T));
    auto load_v = [&](int x, int h, uint32_t (&v)[4][NP][WORDS]) {
        const __amdgpu_buffer_rsrc_t rv = keys_of(V, unit_key(x) + 16 * h, len + 1, D * sizeof(T), 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int off = v_off + (i * D + 16 * PER * j) * static_cast<int>(sizeof(T));
                if constexpr (WORDS == 4) {
                    const auto y = __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, 0);
                    __builtin_memcpy(v[i][j], &y, 16);
                } else {
                    const auto y = __builtin_amdgcn_raw_buffer_load_b64(rv, off, 0, 0);
                    __builtin_memcpy(v[i][j], &y, 8);
                }
            }
    };

    // the statistics' loads first, then the first units (behind them, so that
    // the statistics do not wait for the units)
    const bool own_stats = (a.plane + kChunk - 1) / kChunk <= kStatChunks;
    const int hs = min(tid / 16, G - 1);  // 16 lanes per head
    float2 pr[vz::kPairs];
    if (own_stats) vz::load_pairs(ml_of(a, l, g * G + hs) + it.first, it.n_chunks, tid % 16, pr);
    else pr[0] = a.layer[row_sl * Hq + g * G + hs];
    __builtin_amdgcn_sched_barrier(0);
    Logits sp[DEPTH][NS];
    uint32_t v[DEPTH][2][4][NP][WORDS];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        const int x = min(u, nch - 1);
        load_s(x, sp[u]);
        load_v(x, 0, v[u][0]);
        load_v(x, 1, v[u][1]);
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        const float2 st = own_stats ? vz::merge_pairs(pr, it.n_chunks, tid % 16, ExpRel()) : pr[0];
        if (tid % 16 == 0) s_stat[tid / 16] = tid / 16 < G ? st : make_float2(INFINITY, 1.f);
    }
    __syncthreads();
    const float M = s_stat[hc].x, inv_Z = 1.0f / s_stat[hc].y;

    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // p of four keys of a head per lane; Sum_h p of each key to its place
    auto probabilities = [&](int x, int h, const Logits& p, float (&e)[4]) {
        const int k0 = unit_key(x) + 16 * h;
        e[0] = expf(p.s.x - M);
        e[1] = expf(p.s.y - M);
        e[2] = expf(p.s.z - M);
        e[3] = expf(p.s.w - M);
        float ks[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ks[i] = heads_sum<PACK>(e[i] * inv_Z);
        const float sum = (r16 & 2) ? ((r16 & 1) ? ks[3] : ks[2]) : ((r16 & 1) ? ks[1] : ks[0]);
        if (hc < 4) {
            if (fold) {
                if (k0 + key_off <= len)
                    vz_sel::store_score(sc + k0 + key_off, fmaf(a.gamma, p.old, sum), !RAG && a.ev.cnt);
            } else {
                // (the logits of these keys are in registers: only this wave reads them)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sum), logits_of(x), 4 * (k0 % kChunk + key_off), 0, 0);
            }
        }
    };
    auto product = [&](const uint32_t (&vt)[4][NP][WORDS], const float (&e)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                float f[PER];
                widen<DT, PER>(vt[i][j], f);
#pragma unroll
                for (int k = 0; k < PER; ++k)
                    acc[PER * j + k] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[k], e[i], acc[PER * j + k], 0, 0, 0);
            }
    };
    for (int x0 = 0; x0 < nch; x0 += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int x = x0 + u;
            if (x >= nch || unit_key(x) > len) break;
            const bool more = x + DEPTH < nch;
            float e0[4], e1[4];
            probabilities(x, 0, sp[u][0], e0);
            if constexpr (PACK) {
#pragma unroll
                for (int i = 0; i < 4; ++i) e1[i] = vz::ror16<8>(e0[i]);
            } else {
                probabilities(x, 1, sp[u][NS - 1], e1);
            }
            if (more) load_s(x + DEPTH, sp[u]);
            product(v[u][0], e0);
            if (more) load_v(x + DEPTH, 0, v[u][0]);
            product(v[u][1], e1);
            if (more) load_v(x + DEPTH, 1, v[u][1]);
        }
    }
    // ---- the four waves' outputs, added in wave order ----
    // row 4 q4 + i of tile PER j + k: channel 16 PER j + PER (4 q4 + i) + k
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            s_o[w][r16][16 * PER * (t / PER) + PER * (4 * q4 + i) + t % PER] = acc[t][i];
    __syncthreads();  // ... and every logit of the run has been read
    for (int x = tid; x < G * D; x += kThreads) {
        const int h = x / D, ch = x % D;
        float o = s_o[0][h][ch];
#pragma unroll
        for (int v = 1; v < kWaves; ++v) o += s_o[v][h][ch];
        o /= s_stat[h].y;
        if (rn.n == 1)
            static_cast<T*>(a.out)[(row_sl * Hq + g * G + h) * D + ch] = E::from_f32(o);
        else
            run_out(a, l, it.first + c0, g, G, h)[ch] = o;
    }
    if constexpr (!RAG) {
        if (fold && a.ev.cnt && vz_sel::last_of_layer(a.ev, l, rn.n)) evict_layer<kThreads, T, D>(a, l);
    }
}

// Blocks per sequence behind the fold blocks: one per head, or with one head
// per KV head, where a sequence is always one run, one for the status alone.
__host__ __device__ inline int out_heads(int Hq, int G) { return G == 1 ? 1 : Hq; }

// Fold blocks [0, fold_blocks) of a layer: one chunk's scores, thread = key.
// The blocks after them: one (head, sequence)'s output row from its runs, and
// in a ragged call the sequence's status.
template <int DT, int D, int RAG>
__global__ __launch_bounds__(kChunk) void finish_kernel(const GenericArgs a, int fold_blocks) {
    using E = vz::Elem<DT>;
    const int l = blockIdx.y, t = threadIdx.x;
    const int Hq = a.Hq, Hkv = a.Hkv, G = Hq / Hkv;
    SeqItem it;
    if (static_cast<int>(blockIdx.x) < fold_blocks) {
        int c;
        if (!resolve_chunk<RAG>(a, blockIdx.x, it, c)) return;
        const int key = c * kChunk + t;
        if (key <= it.len) {
            float* const sc = a.score + static_cast<size_t>(l) * a.plane + it.base + key;
            const float old = *sc;
            float sum = 0.f;
    #pragma unroll 4
            for (int g = 0; g < Hkv; ++g) sum += a.S[ws_row(a, l, it.first + c, g * G) * kChunk + t];
            // (zero pad of Eq. (6) for the new slot)
            vz_sel::store_score(sc, fmaf(a.gamma, key < it.len ? old : 0.f, sum), !RAG && a.ev.cnt);
        }
        if constexpr (!RAG) {
            if (a.ev.cnt && vz_sel::last_of_layer(a.ev, l, fold_blocks)) evict_layer<kChunk, typename E::T, D>(a, l);
        }
        return;
    }
    const int ob = static_cast<int>(blockIdx.x) - fold_blocks, heads = out_heads(Hq, G), h = ob % heads, s = ob / heads;
    int first = 0, nc = a.n_chunks;
    if constexpr (RAG) {
        const int st = vz::ragged_decode_status(a.rag, s);
        nc = vz::ragged_chunks(a.rag, s);
        first = vz::ragged_first(s, a.nc_max, [&](int u) { return vz::ragged_chunks(a.rag, u); });
        const bool ok = st == VZ_OK && first >= 0 && first + nc <= a.nc_max;
        if (a.rag.status && h == 0 && l == 0 && t == 0)
            a.rag.status[s] = ok ? VZ_OK : (st != VZ_OK ? st : VZ_ERR_CAPACITY);
        if (!ok) return;
    }
    const Runs rn = runs_of(nc, G);
    if (rn.n == 1 || t >= D) return;
    const int g = h / G, hg = h % G;
    float o = 0.f;
#pragma unroll 8
    for (int r = 0; r < rn.n; ++r) o += run_out(a, l, first + r * rn.step, g, G, hg)[t];
    static_cast<typename E::T*>(a.out)[((static_cast<size_t>(s) * a.L + l) * Hq + h) * D + t] = E::from_f32(o);
}

template <int DT, int D, int RAG>
hipError_t launch(const VzDecodeArgs& v, hipStream_t stream) {
    GenericArgs a{};
    a.q = v.q;
    a.k_new = v.k_new;
    a.v_new = v.v_new;
    a.k_cache = v.k_cache;
    a.v_cache = v.v_cache;
    a.pos = v.pos;
    a.score = v.score;
    a.out = v.out;
    a.Hq = v.Hq;
    a.Hkv = v.Hkv;
    a.L = v.L;
    a.plane = RAG ? v.rag.total : v.cap;
    a.nc_max = static_cast<int32_t>(vz_decode_chunk_rows(a.plane, v.rag.n));
    const size_t rows = static_cast<size_t>(v.L) * a.nc_max * v.Hq;
    a.S = reinterpret_cast<float*>(static_cast<uint8_t*>(v.ws) + vz_decode_hdr_bytes(v.L));
    a.ml = reinterpret_cast<float2*>(a.S + rows * kChunk);
    a.layer = a.ml + rows;
    a.scale = v.sm_scale > 0.f ? v.sm_scale : 1.0f / sqrtf(static_cast<float>(D));
    a.gamma = v.gamma;
    a.rag = v.rag;
    const int G = v.Hq / v.Hkv, seqs = RAG ? v.rag.n : 1;
    int chunks = a.nc_max, runs = a.nc_max;  // grid extents per layer and KV head
    if (!RAG) {
        a.len = v.len;
        a.next_pos = v.next_pos;
        a.n_chunks = chunks = v.len / kChunk + 1;  // of len + 1 keys
        runs = runs_of(chunks, G).n;
        // arrival counters: in the layer statistics' place, or, where those are
        // used, in a pair of each layer's head 0 past the sequence's chunks
        // (whose distance, a layer's pairs, passes 2^31 at terabytes of cache)
        const bool own_stats = (a.plane + kChunk - 1) / kChunk <= kStatChunks;
        if (v.ev)
            a.ev = vz_sel::EvictOne{reinterpret_cast<uint64_t*>(own_stats ? a.layer : a.ml + a.nc_max - 1),
                                    own_stats ? a.Hq : a.Hq * a.nc_max, v.ev_budget, v.ev_sink, v.ev_M};
    }
    if (G <= 8)
        hipLaunchKernelGGL((logits_kernel<DT, D, RAG, true>), dim3(chunks, a.L, a.Hkv), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((logits_kernel<DT, D, RAG, false>), dim3(chunks, a.L, a.Hkv), dim3(kThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((a.plane + kChunk - 1) / kChunk > kStatChunks) {
        hipLaunchKernelGGL((stats_kernel<(RAG != 0)>), dim3((a.Hq + 15) / 16, a.L, seqs), dim3(kThreads), 0, stream, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (G <= 8)
        hipLaunchKernelGGL((values_kernel<DT, D, RAG, true>), dim3(runs, a.L, a.Hkv), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((values_kernel<DT, D, RAG, false>), dim3(runs, a.L, a.Hkv), dim3(kThreads), 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int folds = a.Hkv > 1 ? chunks : 0;  // one KV head: folded by the values kernel
    const int outs = RAG || runs > 1 ? out_heads(a.Hq, G) * seqs : 0;
    if (folds + outs == 0) return hipSuccess;
    hipLaunchKernelGGL((finish_kernel<DT, D, RAG>), dim3(folds + outs, a.L), dim3(kChunk), 0, stream, a, folds);
    return hipGetLastError();
}

template <int DT, int D>
hipError_t launch_any(const VzDecodeArgs& v, hipStream_t stream) {
    if (v.rag.n > kManySeqs) return launch<DT, D, 2>(v, stream);
    return v.rag.n > 0 ? launch<DT, D, 1>(v, stream) : launch<DT, D, 0>(v, stream);
}

}  // namespace

hipError_t vz_launch_decode_generic(const VzDecodeArgs& a, hipStream_t stream) {
    if (a.dtype == VZ_BF16 && a.d == 128) return launch_any<VZ_BF16, 128>(a, stream);
    if (a.dtype == VZ_BF16 && a.d == 64) return launch_any<VZ_BF16, 64>(a, stream);
    if (a.dtype == VZ_F32 && a.d == 128) return launch_any<VZ_F32, 128>(a, stream);
    if (a.dtype == VZ_F32 && a.d == 64) return launch_any<VZ_F32, 64>(a, stream);
    return hipErrorInvalidValue;
}
