// Decode step (Sec. 3.1 Eq. 1-2, Sec. 3.2.2 Eq. 6) for bfloat16 caches with
// d = 128 and at most 8 query heads per KV head, chunked path.  The attend
// kernel streams the cache once and leaves per-chunk partial results in the
// workspace; a finishing launch (or an output and a fold launch) merges them
// into the output rows and the decayed scores.  No workgroup ever waits for
// another.  Calls with enough (layer, KV head) items go to the whole-range
// path (decode_range.hip) instead.
//
// Attend kernel: work item = (layer, key chunk of <= 128 keys, KV head), a
// workgroup of four waves, one 32-key tile each (the query rows and the K
// and V tiles of a wave are requested at once: one memory round trip per
// chunk, and both tiles are used from registers).
//   logits  S^T = K Q^T with v_mfma_f32_16x16x32_bf16 (M = 16 keys, N = 16
//           query-head columns of which n_q/n_kv <= 8 are used, K = 32
//           channels), K rows loaded in the A-operand layout.  The logits
//           of the odd 16-key half of a tile are moved into the unused head
//           columns 8..15 (DPP row rotate by 8), so 32 keys x 8 heads take 4
//           registers per lane.
//   stats   per wave and head the max m_w and the sum of exp2 relative to it.
//   P V     O^T = V^T P^T with the same instruction over the tile's 32 keys:
//           the A operands are gathered from whole V rows by byte permutes, P
//           (bfloat16) needs one row rotate.
//   merge   at the one barrier the waves' outputs are rescaled to the chunk's
//           max m_c and added in wave order; (m_c, l_c), O_c and p~ = exp2(s -
//           m_c) per key (both bfloat16) go to the workspace.
// Output blocks: per (head, layer), the output row merged from the chunk
// partials.  Fold blocks: per (chunk, layer), the chunk's scores A[j] = gamma
// A[j] + sum_h p_hj from p~ and one factor per head; in a generation step with
// one eviction due the layer's last fold block does it.
#include <algorithm>
#include <atomic>
#include <random>
#include <type_traits>

#include "decode_mfma.h"
#include "select.h"

namespace {

using namespace vz_mfma;

// Decode workspace header: 256 reserved bytes (a ragged call keeps its table
// sizes there), then one arrival counter per layer (whole-range path, zero
// after every call), padded to 256 bytes.
constexpr size_t kHeaderBytes = 256;

// Per-chunk partial results in the workspace, after the header:
//   ml [L][Hq][nc_max]        float2     chunk max m_c and sum l_c of exp2, per head (a head's chunks
//                                        side by side: the finishing kernels read them 16 lanes at a time)
//   o  [L][nc_max][Hq][D]     bfloat16   O_c relative to m_c
//   p  [L][nc_max][Hq][CHUNK] bfloat16   p~ = exp2(s - m_c) per key of the chunk
//   layer [S][L][Hq]          float2     the layer's max M and 1 / sum S, per head
//                                        (S = sequences of the call; calls of two
//                                        finishing launches only: with one, a generation
//                                        step's arrival counters, Hq apart)
template <typename B>
struct PartialsT {
    using F2 = typename std::conditional<std::is_const<B>::value, const float2, float2>::type;
    using U16 = typename std::conditional<std::is_const<B>::value, const uint16_t, uint16_t>::type;
    F2* ml;
    U16* o;
    U16* p;
    F2* layer;
    __device__ PartialsT(B* ws, int hdr_bytes, int L, int nc_max, int Hq) {
        const size_t n = static_cast<size_t>(L) * nc_max * Hq;
        ml = reinterpret_cast<F2*>(ws + hdr_bytes);
        o = reinterpret_cast<U16*>(ml + n);
        p = o + n * D;
        layer = reinterpret_cast<F2*>(p + n * CHUNK);
    }
};
using Partials = PartialsT<uint8_t>;
using ConstPartials = PartialsT<const uint8_t>;

using vz::SeqItem;
using vz::ragged_chunks;
static_assert(CHUNK == vz::kChunk, "one chunk size");

struct Exp2Rel {
    __device__ __forceinline__ float operator()(float x, float m) const { return x == -INFINITY ? 0.f : exp2f(x - m); }
};
// The weights of the chunks in a head's sums, where the chunk of the max has
// weight 1 and a sum of exp of at least 1: the instruction alone, whose flush
// of weights below 2^-126 is far below the sums' last bit.
struct Exp2Weight {
    __device__ __forceinline__ float operator()(float x, float m) const { return __builtin_amdgcn_exp2f(x - m); }
};

// Flat chunk f of a call: false when it holds no work.
template <bool RAG>
__device__ __forceinline__ bool resolve_chunk(const FusedArgs& a, int f, SeqItem& it, int& c) {
    if constexpr (RAG) {
        return vz::locate_ragged_chunk(a.rag, a.nc_max, f, it, c);
    } else {
        if (f >= a.n_chunks) return false;
        it.s = 0;
        it.len = a.len;
        it.next_pos = a.next_pos;
        it.n_chunks = a.n_chunks;
        it.first = 0;
        it.base = 0;
        c = f;
    }
    return true;
}

// Attend kernel: work item = (layer, chunk, KV head), a workgroup of SPLIT_W
// waves in which wave w owns keys [VT w, VT w + VT) of the chunk.  Each wave
// requests its query rows and its K and V tile (16 KB) before anything else,
// so a chunk costs one memory round trip, and a one-layer call over 8k keys
// spreads its 16 MB over 260 workgroups.  Both tiles come in the MFMA operand
// layouts and stay in registers: the softmax is relative to the wave's own max
// until the waves meet once, at the end, where their outputs are rescaled to
// the chunk's max and summed in wave order.  A one-layer call is a launch
// (1.7 us), its 16.8 MB (3.8 us for a kernel of the same loads and nothing
// else) and this arithmetic behind the last loads, 1.9 us with the stores: per
// layer of a 48-layer graph at 8,200 keys, with the finishing launch and a
// caller's kernel, 14.9 -> 13.4 us (V through LDS, three barriers and the
// sequence search by shuffles before).
// (Launch bounds: four workgroups per CU, 128 registers per lane; the MFMA
// accumulators then live in ordinary vector registers.)
constexpr int SPLIT_W = CHUNK / VT;  // waves per chunk: one 32-key tile each
template <int NW, bool RAG>
__global__ __launch_bounds__(64 * SPLIT_W, 4) void decode_attend_kernel(const FusedArgs a) {
    constexpr int OS = D + 4;  // padded LDS row of a wave's partial output (floats)
    __shared__ __attribute__((aligned(16))) float s_o[SPLIT_W][GMAX][OS];
    __shared__ float s_m[SPLIT_W][GMAX], s_l[SPLIT_W][GMAX];
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int q4 = lane >> 4, r16 = lane & 15;
    const int hi = r16 >> 3, hh = r16 & 7;
    const int Hq = a.Hq, nc_max = a.nc_max;
    const int G = Hq / NW;
    // item = (chunk item, KV head), KV head fastest; a ragged call's layers
    // are on grid y; a single sequence's chunk items are its full chunks of
    // every layer first, then the short remainders
    const int g = static_cast<int>(blockIdx.x) % NW;
    const int ci = static_cast<int>(blockIdx.x) / NW;
    int l, f;
    if constexpr (RAG) {
        l = blockIdx.y;
        f = ci;
    } else {
        const int n_full = (a.len + 1) / CHUNK;
        if (a.L == 1) {
            l = 0;
            f = ci;
        } else if (ci < a.L * n_full) {
            l = ci / n_full;
            f = ci - l * n_full;
        } else {
            l = ci - a.L * n_full;
            f = n_full;
        }
    }
    SeqItem it;
    int c;
    if (!resolve_chunk<RAG>(a, f, it, c)) return;
    const int len = it.len, T = len + 1;
    const int k_begin = chunk_begin(c);
    const int nk = chunk_keys(c, T);
    const int kw0 = k_begin + VT * w;  // the wave's first key
    const int rows = min(VT, max(nk - VT * w, 0));
    const size_t head_base = ((static_cast<size_t>(l) * NW + g) * a.plane + it.base) * D;
    uint16_t* Kh = a.k_cache + head_base;
    uint16_t* Vh = a.v_cache + head_base;
    const size_t row_sl = static_cast<size_t>(it.s) * a.L + l;

    float sp[4] = {0.f, 0.f, 0.f, 0.f}, m_w = -INFINITY;  // the wave's p (4 keys of a head per lane) and max
    if (rows > 0) {
        // Eq. (1): the wave whose keys hold slot len (row rr of its tile) loads
        // its KV head's new K and V rows with its other loads, puts them into its
        // tile registers in place of the cache's old row once the tiles have
        // landed, and only then writes them to the cache (and KV head 0 the
        // position), so that none of the chunk's loads waits behind a write.
        // Lane (r16, q4) holds K channels 8 (q4 + 4 s) .. + 7 of its K rows and V
        // channels 8 r16 .. + 7 of its V rows (the tile layouts below).
        const int rr = len - kw0;
        if (!RAG && a.ev != 0 && f == 0 && g == 0 && tid == 0) a.cnt[l * static_cast<size_t>(a.cnt_stride)] = 0;  // counted by the finishing launch
        const bool writer = rr >= 0 && rr < VT;  // wave-uniform
        uint4 kn_row[KSTEPS], vn_row;
        if (writer) {
            const uint16_t* kn = a.k_new + (row_sl * NW + g) * D;
            const uint16_t* vn = a.v_new + (row_sl * NW + g) * D;
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) kn_row[s] = *reinterpret_cast<const uint4*>(kn + 8 * (q4 + 4 * s));
            vn_row = *reinterpret_cast<const uint4*>(vn + 8 * r16);
        }

        // The query rows first, so that the logits wait for them and the K tile
        // only, not for the V tile behind them.  One descriptor over the KV
        // head's G query rows: lanes of head columns r16 >= G read past it and
        // get zeros, with no memory access.
        uint4 qv[KSTEPS];
        {
            const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint16_t*>(a.q + (row_sl * Hq + g * G) * D), 0, __builtin_amdgcn_readfirstlane(G * D * 2),
                kBufferDword3);
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(rq, (r16 * D + 8 * q4 + 32 * s) * 2, 0, 0);
                __builtin_memcpy(&qv[s], &v, 16);
            }
        }

        // both tiles requested at once; rows past the chunk read as zero without
        // touching memory (bounded scalar descriptors).  K in the MFMA A-operand
        // layout: register m = 4 ti + s holds bytes 16 (q4 + 4 s) .. + 15 of row
        // 16 ti + r16.  V whole rows at a time, 16 bytes of four rows per lane and
        // tile half: register m = 4 ti + i holds channels 8 r16 .. + 7 of row
        // 16 ti + 4 q4 + i, which are the lane's share of eight A operands (V^T,
        // channel slot r16 of output tile e: channel 8 r16 + e) for those keys.
        const int lane_off_k = r16 * (D * 2) + 16 * q4;
        const int lane_off_v = 4 * q4 * (D * 2) + 16 * r16;
        uint4 kt[8], vt[8];
        {
            // (the byte bound taken through readfirstlane keeps the descriptors in
            // scalar registers: a bound left in a vector register makes the
            // compiler wrap every load in a loop over the lanes' descriptors)
            const int nbytes = __builtin_amdgcn_readfirstlane(rows * D * 2);
            const __amdgpu_buffer_rsrc_t rk =
                __builtin_amdgcn_make_buffer_rsrc(Kh + static_cast<size_t>(kw0) * D, 0, nbytes, kBufferDword3);
            const __amdgpu_buffer_rsrc_t rv =
                __builtin_amdgcn_make_buffer_rsrc(Vh + static_cast<size_t>(kw0) * D, 0, nbytes, kBufferDword3);
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(rk, lane_off_k + (m >> 2) * 16 * (D * 2) + (m & 3) * 64,
                                                                     0, 0);
                __builtin_memcpy(&kt[m], &v, 16);
            }
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const auto v =
                    __builtin_amdgcn_raw_buffer_load_b128(rv, lane_off_v + (16 * (m >> 2) + (m & 3)) * (D * 2), 0, 0);
                __builtin_memcpy(&vt[m], &v, 16);
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // every load above is issued before the first wait

        if (writer && r16 == (rr & 15)) {  // the new K row: row 16 ti + r16 of registers 4 ti .. 4 ti + 3
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
                if (ti == rr >> 4)
#pragma unroll
                    for (int s = 0; s < KSTEPS; ++s) kt[4 * ti + s] = kn_row[s];
        }

        // ---- logits of the wave's 32 keys: S^T = K Q^T ----
        f32x4 acc[2];
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
            acc[ti] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s)
                acc[ti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kt[4 * ti + s]), as_bf16x8(qv[s]), acc[ti], 0,
                                                                  0, 0);
        }
        // packed: head column r16 < 8 keeps the even half's logits, column r16 =
        // 8 + hh takes the odd half's of head hh
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float odd = ror8(acc[1][i]);
            const float v = hi ? odd : acc[0][i];
            const int key = VT * w + 16 * hi + 4 * q4 + i;  // within the chunk
            sp[i] = (key < nk) ? v * a.scale_log2 : -INFINITY;
        }
        // ---- p relative to the wave's max, per head ----
        m_w = fmaxf(fmaxf(sp[0], sp[1]), fmaxf(sp[2], sp[3]));
        m_w = vz::rows_max(m_w);
        m_w = fmaxf(m_w, ror8(m_w));
        const float ref = finite_ref(m_w);
        float l_w = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sp[i] = exp2f(sp[i] - ref);
            l_w += sp[i];
        }
        l_w = vz::rows_sum(l_w);
        l_w += ror8(l_w);
        if (q4 == 0 && hi == 0) {
            s_m[w][hh] = m_w;
            s_l[w][hh] = l_w;
        }
        // B operand P^T: columns 0..7 the even half's keys, then the odd half's
        // (columns 8..15 hold the halves the other way round: outputs not used)
        const uint32_t p01 = pack_bf16x2(sp[0], sp[1]), p23 = pack_bf16x2(sp[2], sp[3]);
        const bf16x8_t pb = as_bf16x8(make_uint4(p01, p23, ror8_u32(p01), ror8_u32(p23)));

        if (writer) {
            if (q4 == ((rr >> 2) & 3)) {  // the new V row: row 16 ti + 4 q4 + i of register 4 ti + i
#pragma unroll
                for (int m = 0; m < 8; ++m)
                    if (m == 4 * (rr >> 4) + (rr & 3)) vt[m] = vn_row;
            }
            // the new rows into the cache, after every load of the wave (a plane's
            // element offsets pass 2^31 at 2^24 slots)
            const size_t at = static_cast<size_t>(len) * D;
            if (r16 == (rr & 15)) {
#pragma unroll
                for (int s = 0; s < KSTEPS; ++s) *reinterpret_cast<uint4*>(Kh + at + 8 * (q4 + 4 * s)) = kn_row[s];
            }
            if (q4 == ((rr >> 2) & 3)) *reinterpret_cast<uint4*>(Vh + at + 8 * r16) = vn_row;
            if (g == 0 && lane == 0) a.pos[static_cast<size_t>(l) * a.plane + it.base + len] = it.next_pos;
        }

        // ---- O^T = V^T P^T over the wave's keys ----
        // Output tile e takes channel 8 slot + e of each of the 16 channel slots:
        // its A operand is element e of the lane's eight V pieces (keys 4 q4 + i,
        // then 16 + 4 q4 + i, as in pb), gathered by byte permutes.
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        f32x4 oacc[DTILES];
#pragma unroll
        for (int e = 0; e < DTILES; ++e) {
            uint32_t x[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint32_t words[4] = {vt[m].x, vt[m].y, vt[m].z, vt[m].w};
                x[m] = words[e / 2];
            }
            constexpr uint32_t kLow = 0x05040100u, kHigh = 0x07060302u;  // halves of (second, first) word
            uint32_t av[4];
#pragma unroll
            for (int y = 0; y < 4; ++y) av[y] = __builtin_amdgcn_perm(x[2 * y + 1], x[2 * y], (e & 1) ? kHigh : kLow);
            oacc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(make_uint4(av[0], av[1], av[2], av[3])), pb, zero,
                                                              0, 0, 0);
        }
        // lane: head r16, channels 8 (4 q4 + i) + e
        if (r16 < G) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < DTILES; e += 4)
                    *reinterpret_cast<float4*>(&s_o[w][r16][8 * (4 * q4 + i) + e]) =
                        make_float4(oacc[e][i], oacc[e + 1][i], oacc[e + 2][i], oacc[e + 3][i]);
        }
    } else {
        // past the chunk's keys: nothing to add.  (At 65 chunks x 4 KV heads on
        // 256 CUs four CUs hold two workgroups and end last; the short last
        // chunk's idle waves took their issue slots: 668 -> 645 us per token.)
        if (lane < GMAX) {
            s_m[w][lane] = -INFINITY;
            s_l[w][lane] = 0.f;
        }
        for (int i = lane; i < GMAX * OS; i += vz::kWave) (&s_o[w][0][0])[i] = 0.f;
    }
    __syncthreads();

    // ---- partial results of (chunk, head): (m_c, l_c), O_c and p~ ----
    Partials part(a.ws, a.hdr_bytes, a.L, nc_max, Hq);
    const int pbase = (l * nc_max + it.first + c) * Hq + g * G;  // < 2^31 (checked on the host)
    auto chunk_max = [&](int h) { return fmaxf(fmaxf(s_m[0][h], s_m[1][h]), fmaxf(s_m[2][h], s_m[3][h])); };
    static_assert(SPLIT_W == 4, "four waves' maxima");
    {
        // p~ = p rescaled to the chunk's max, 4 keys of a head per lane
        const float f = exp2f(m_w - finite_ref(chunk_max(hh)));
        if (hh < G && rows > 0)
            *reinterpret_cast<uint2*>(part.p + static_cast<size_t>(pbase + hh) * CHUNK + VT * w + 16 * hi + 4 * q4) =
                make_uint2(pack_bf16x2(sp[0] * f, sp[1] * f), pack_bf16x2(sp[2] * f, sp[3] * f));
    }
    {
        // 4 channels per thread, whole output rows per head
        const int h = tid >> 5, c4 = 4 * (tid & 31);
        if (h < G) {
            const float m_c = chunk_max(h), ref = finite_ref(m_c);
            float o[4] = {0.f, 0.f, 0.f, 0.f}, lc = 0.f;
#pragma unroll
            for (int v = 0; v < SPLIT_W; ++v) {
                const float f = Exp2Weight()(s_m[v][h], ref);
                const float4 x = *reinterpret_cast<const float4*>(&s_o[v][h][c4]);
                o[0] = fmaf(x.x, f, o[0]);
                o[1] = fmaf(x.y, f, o[1]);
                o[2] = fmaf(x.z, f, o[2]);
                o[3] = fmaf(x.w, f, o[3]);
                lc = fmaf(s_l[v][h], f, lc);
            }
            *reinterpret_cast<uint2*>(part.o + static_cast<size_t>(pbase + h) * D + c4) =
                make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
            if (c4 == 0) part.ml[(l * Hq + g * G + h) * nc_max + it.first + c] = make_float2(m_c, lc);
        }
    }
}

// ---- finishing: merge of the chunk partials ----
// Sums use explicit fused multiply-adds, so the bits do not depend on how the
// compiler contracts each kernel (the single-sequence and ragged calls, and
// the two forms of the finishing launches, give the same bits).
constexpr int OUT_THREADS = 256;
constexpr int OUT_ROWS = OUT_THREADS / 16;  // row groups
constexpr int OUT_BATCH = vz::kPairs;       // chunks per row group and round
static_assert(OUT_ROWS == 16, "a row group per lane of a DPP row");

// Output row of head h of (layer l, sequence s) by a whole block: thread t
// owns channels 8 (t % 16) .. + 7 of the rows of chunks t / 16, t / 16 + 16,
// ...; o = sum_c O_c exp2(m_c - M) / S with the head's (M, S), which every
// 16-lane row of the block forms itself (no barrier before the weights), so
// the weighted rows are independent of one another; the 16 row groups are
// summed in registers within a wave and through LDS across the waves.
struct OutLoads {
    float2 pr[vz::kPairs];   // the statistics' pairs (lane t % 16)
    float m[OUT_BATCH];      // the maxima of the thread's own chunks
    uint4 x[OUT_BATCH];      // their row pieces
};
__device__ __forceinline__ void out_load(const float2* ml, const uint16_t* po, int Hq, int c0, int n_load, float* m,
                                         uint4* x) {
#pragma unroll
    for (int k = 0; k < OUT_BATCH; ++k) {  // rows clamped (every load in bounds), masked later
        m[k] = -INFINITY;
        x[k] = make_uint4(0, 0, 0, 0);
        if (OUT_ROWS * k >= n_load) continue;  // uniform
        const int cc = min(c0 + OUT_ROWS * k, n_load - 1);
        m[k] = ml[cc].x;
        x[k] = *reinterpret_cast<const uint4*>(po + static_cast<size_t>(cc) * Hq * D);
    }
}
__device__ __forceinline__ void out_add(const float* m, const uint4* x, int c0, int n_chunks, float M, float (&acc)[8]) {
#pragma unroll
    for (int k = 0; k < OUT_BATCH; ++k) {
        if (OUT_ROWS * k >= n_chunks) break;  // uniform
        const float wgt = Exp2Weight()(c0 + OUT_ROWS * k < n_chunks ? m[k] : -INFINITY, M);
        float f[8];
        vz::unpack16<VZ_BF16>(x[k], f);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = fmaf(wgt, c0 + OUT_ROWS * k < n_chunks ? f[i] : 0.f, acc[i]);
    }
}
__device__ __forceinline__ void out_store(const FusedArgs& a, int h, int l, int s, float inv_S, float (&acc)[8]) {
    constexpr int WAVES = OUT_THREADS / vz::kWave;
    __shared__ __attribute__((aligned(16))) float s_acc[WAVES][D];
    const int t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = vz::rows_sum(acc[i]);
    if (t % vz::kWave < 16) {
        float* const d = &s_acc[t / vz::kWave][8 * (t % 16)];
        *reinterpret_cast<float4*>(d) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        *reinterpret_cast<float4*>(d + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
    __syncthreads();
    if (t < D) {
        float o = s_acc[0][t];
#pragma unroll
        for (int v = 1; v < WAVES; ++v) o += s_acc[v][t];
        a.out[((static_cast<size_t>(s) * a.L + l) * a.Hq + h) * D + t] = vz::f32_to_bf16(o * inv_S);
    }
}

// Output block of (head h, layer l, sequence s); store_layer: also the head's
// (M, 1 / S) for the fold kernel.  ONE (a call of one sequence whose planes
// hold at most vz::kPairChunks chunks): its chunk rows start at row 0, so the
// partial results' loads (rows clamped to the layer's) go out before the
// sequence's values arrive.  In a ragged call the block of head 0 of layer 0
// reports the sequence's status.
template <bool RAG, bool ONE>
__device__ void output_block(const FusedArgs& a, int h, int l, int s, bool store_layer) {
    const int t = threadIdx.x, Hq = a.Hq;
    const int rg = t / 16, c8 = 8 * (t % 16);
    Partials part(a.ws, a.hdr_bytes, a.L, a.nc_max, Hq);
    const float2* const ml = part.ml + (static_cast<size_t>(l) * Hq + h) * a.nc_max;
    const uint16_t* const po = part.o + (static_cast<size_t>(l) * a.nc_max * Hq + h) * D + c8;
    OutLoads ld;
    auto load = [&](int first, int n_load) {
        vz::load_pairs(ml + first, n_load, t % 16, ld.pr);
        out_load(ml + first, po + static_cast<size_t>(first) * Hq * D, Hq, rg, n_load, ld.m, ld.x);
    };
    if constexpr (ONE) {
        load(0, RAG ? a.nc_max : a.n_chunks);
        __builtin_amdgcn_sched_barrier(0);  // every load is issued before the first wait
    }
    int first = 0, n_chunks = a.n_chunks;
    if constexpr (RAG) {
        // the sequence's own values and the earlier sequences' chunk counts
        // are loaded side by side (one round of loads)
        const int st = vz::ragged_decode_status(a.rag, s);
        if constexpr (!ONE) first = vz::ragged_first(s, a.nc_max, [&](int u) { return ragged_chunks(a.rag, u); });
        n_chunks = st == VZ_OK ? (a.rag.len[s] + CHUNK) / CHUNK : 0;
        const bool ok = st == VZ_OK && first >= 0 && first + n_chunks <= a.nc_max;
        if (a.rag.status && h == 0 && l == 0 && t == 0) a.rag.status[s] = ok ? VZ_OK : (st != VZ_OK ? st : VZ_ERR_CAPACITY);
        if (!ok) return;
    }
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    float2 stats;
    if (ONE || n_chunks <= vz::kPairChunks) {
        if constexpr (!ONE) {
            load(first, n_chunks);
            __builtin_amdgcn_sched_barrier(0);
        }
        stats = vz::merge_pairs(ld.pr, n_chunks, t % 16, Exp2Weight());
        out_add(ld.m, ld.x, rg, n_chunks, stats.x, acc);
    } else {
        // the max by the whole block, so that only the sum is a chain of loads
        // through all chunks (2,344 chunks: the kernel 33.4 -> 27 us)
        __shared__ float s_max[OUT_THREADS / vz::kWave];
        float m = -INFINITY;
#pragma unroll 8
        for (int c = t; c < n_chunks; c += OUT_THREADS) m = fmaxf(m, ml[first + c].x);
        m = vz::rows_max(vz::row16_max(m));
        if (t % vz::kWave == 0) s_max[t / vz::kWave] = m;
        __syncthreads();
#pragma unroll
        for (int v = 0; v < OUT_THREADS / vz::kWave; ++v) m = fmaxf(m, s_max[v]);
        stats = make_float2(m, vz::merge_sum(ml + first, n_chunks, t % 16, m, Exp2Weight()));
        for (int c0 = rg; c0 - rg < n_chunks; c0 += OUT_ROWS * OUT_BATCH) {
            out_load(ml + first, po + static_cast<size_t>(first) * Hq * D, Hq, c0, n_chunks, ld.m, ld.x);
            out_add(ld.m, ld.x, c0, n_chunks, stats.x, acc);
        }
    }
    const float inv_S = 1.0f / stats.y;
    if (store_layer && t == 0) part.layer[(static_cast<size_t>(s) * a.L + l) * Hq + h] = make_float2(stats.x, inv_S);
    out_store(a, h, l, s, inv_S, acc);
}

// Fold of one chunk's scores, Eq. (6), by a block of OUT_THREADS threads:
// A[j] = gamma A[j] + sum_h p~_hj f_h with f_h = exp2(m_c,h - M_h) / S_h (the
// new slot starts from 0).  Wave w adds its quarter of the heads for every key
// of the chunk, two keys per lane, and the four waves' sums meet in LDS.  The
// p~ loads (rows of CHUNK entries; those past the chunk's keys hold anything, a
// lane's two keys stay apart and the store is masked) and the old score's are
// issued before the factors are known.
constexpr int FOLD_HEADS = 16;  // heads per wave: Hq <= Hkv * GMAX with Hkv <= 8
struct FoldLoads {
    uint32_t p[FOLD_HEADS];
    float old;
};
__device__ __forceinline__ int fold_heads_per_wave(int Hq) { return (Hq + 3) / 4; }
// (chunk_row: the chunk's row of the workspace arrays; one descriptor over its
// Hq rows, so a load is an immediate offset from one address, and heads past
// the last read as zero)
__device__ __forceinline__ void fold_load(const ConstPartials& part, size_t chunk_row, int Hq, FoldLoads& ld) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / vz::kWave), lane = threadIdx.x % vz::kWave;
    const int hpw = fold_heads_per_wave(Hq);
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(part.p + chunk_row * Hq * CHUNK), 0, Hq * CHUNK * 2, kBufferDword3);
    const int off = w * hpw * CHUNK * 2 + 4 * lane;
#pragma unroll
    for (int q = 0; q < FOLD_HEADS; ++q) {
        if (q % 8 == 0 && q >= hpw) break;  // wave-uniform
        ld.p[q] = __builtin_amdgcn_raw_buffer_load_b32(rp, off + q * CHUNK * 2, 0, 0);
    }
}
__device__ __forceinline__ void fold_finish(const FusedArgs& a, const FoldLoads& ld, const float* s_f, float* sc, int Hq,
                                            int nk, bool new_key, bool coherent) {
    __shared__ float s_sum[OUT_THREADS / vz::kWave][CHUNK];
    const int t = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(t / vz::kWave), lane = t % vz::kWave;
    const int hpw = fold_heads_per_wave(Hq);
    float x = 0.f, y = 0.f;
#pragma unroll
    for (int q = 0; q < FOLD_HEADS; ++q) {
        if (q < hpw && w * hpw + q < Hq) {
            const float f = s_f[w * hpw + q];
            x = fmaf(bf16_lo(ld.p[q]), f, x);
            y = fmaf(bf16_hi(ld.p[q]), f, y);
        }
    }
    *reinterpret_cast<float2*>(&s_sum[w][2 * lane]) = make_float2(x, y);
    __syncthreads();
    if (t < nk) {
        float acc = s_sum[0][t];
#pragma unroll
        for (int v = 1; v < OUT_THREADS / vz::kWave; ++v) acc += s_sum[v][t];
        // (zero pad of Eq. (6) for the new slot)
        vz_sel::store_score(sc, fmaf(a.gamma, new_key ? 0.f : ld.old, acc), coherent);
    }
}

// Two launches, for the calls that finish_in_one_launch refuses: the output
// kernel, one block per (head, layer, sequence), then the fold kernel, one
// block per (chunk, layer), with the statistics the output kernel stored.
// (Seven waves per SIMD: left alone the compiler takes 93 registers for the
// unrolled loop over many chunks and five, and a batch of 300 short sequences,
// 8 layers, costs 260 us instead of 231.)
template <bool RAG>
__global__ __launch_bounds__(OUT_THREADS, 7) void decode_output_kernel(const FusedArgs a) {
    output_block<RAG, false>(a, blockIdx.x, blockIdx.y, blockIdx.z, true);
}
template <bool RAG>
__global__ __launch_bounds__(OUT_THREADS) void decode_fold_kernel(const FusedArgs a) {
    __shared__ float s_f[8 * GMAX];
    const int l = blockIdx.y, t = threadIdx.x, Hq = a.Hq;
    SeqItem it;
    int c;
    if (!resolve_chunk<RAG>(a, blockIdx.x, it, c)) return;
    const ConstPartials part(a.ws, a.hdr_bytes, a.L, a.nc_max, Hq);
    const int nk = chunk_keys(c, it.len + 1), tk = min(t, nk - 1);
    float* const sc = a.score + static_cast<size_t>(l) * a.plane + it.base + chunk_begin(c) + tk;
    FoldLoads ld;
    const float2 gl = part.layer[(static_cast<size_t>(it.s) * a.L + l) * Hq + min(t, Hq - 1)];
    const float m_c = part.ml[(static_cast<size_t>(l) * Hq + min(t, Hq - 1)) * a.nc_max + it.first + c].x;
    fold_load(part, static_cast<size_t>(l) * a.nc_max + it.first + c, Hq, ld);
    ld.old = *sc;
    if (t < Hq) s_f[t] = Exp2Rel()(m_c, gl.x) * gl.y;
    __syncthreads();
    fold_finish(a, ld, s_f, sc, Hq, nk, chunk_begin(c) + tk == it.len, false);
}

// One launch (see finish_in_one_launch).  Blocks [0, n_chunks)
// of a layer are fold blocks: one per chunk, each forms every head's layer
// statistics itself from its sequence's chunk pairs (16 lanes per head, four
// heads per wave at a time, in registers), with the output blocks' arithmetic
// and order, then folds its chunk's keys.  The blocks after them are output
// blocks, one per (head, sequence), run beside the fold blocks.  The
// recomputation reads n_chunks x Hq pairs per fold block.  Of its 3.5 us above
// an empty kernel (65 chunks, in a graph) 2.5 us are the loads of what the
// attend kernel has just written; addresses are immediate offsets from a few
// descriptors, because at one wave per SIMD each instruction before the loads
// costs its own 2 ns.
constexpr int FINISH_BATCH_CHUNKS = 640;
constexpr int FINISH_BATCH_BLOCKS = 2048;
constexpr int FINISH_ROUNDS = 8 * GMAX / 16;  // of 16 heads
template <bool RAG>
__global__ __launch_bounds__(OUT_THREADS) void decode_finish_kernel(const FusedArgs a) {
    __shared__ float s_f[8 * GMAX];
    const int t = threadIdx.x, l = blockIdx.y, Hq = a.Hq;
    // One sequence (a single-sequence call, or a ragged call of one): its
    // chunk rows start at row 0 of the layer and a fold block's chunk is row
    // blockIdx.x, so every partial-result load is issued before the
    // sequence's values are known (rows clamped to the layer's rows, values
    // masked once they are): one round of loads instead of two.
    const bool one = !RAG || a.rag.n == 1;
    if (static_cast<int>(blockIdx.x) >= a.n_chunks) {
        const int ob = static_cast<int>(blockIdx.x) - a.n_chunks;
        if (one)
            output_block<RAG, true>(a, ob % Hq, l, 0, false);
        else
            output_block<RAG, false>(a, ob % Hq, l, ob / Hq, false);
        return;
    }
    const ConstPartials part(a.ws, a.hdr_bytes, a.L, a.nc_max, Hq);
    float2 pr[FINISH_ROUNDS][vz::kPairs];
    float m_own[FINISH_ROUNDS];
    FoldLoads ld;
    const int tk = t < CHUNK ? t : 0;
    // (one descriptor over the layer's pairs: a load is an immediate offset
    // from the lane's address, and nothing needs clamping)
    auto load = [&](int first, int n_load, int row) {
        const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float2*>(part.ml + static_cast<size_t>(l) * Hq * a.nc_max), 0,
            __builtin_amdgcn_readfirstlane(Hq * a.nc_max * 8), kBufferDword3);
#pragma unroll
        for (int u = 0; u < FINISH_ROUNDS; ++u) {
            if (16 * u >= Hq) break;  // uniform
            const int head = (16 * u + t / 16) * a.nc_max;
            const int off = 8 * (head + first + t % 16);
#pragma unroll
            for (int k = 0; k < vz::kPairs; ++k) {
                pr[u][k] = make_float2(-INFINITY, 0.f);
                if (16 * k < n_load)
                    pr[u][k] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rm, off + 128 * k, 0, 0));
            }
            m_own[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, 8 * (head + row), 0, 0));
        }
        fold_load(part, static_cast<size_t>(l) * a.nc_max + row, Hq, ld);
    };
    SeqItem it;
    int c;
    if (one) {
        load(0, RAG ? a.nc_max : a.n_chunks, blockIdx.x);
        // the score of key tk of chunk blockIdx.x for a sequence at slot 0 (a
        // single-sequence call, or the one slot of a decode loop), with the
        // other loads; another base loads it again once the values are in
        ld.old = a.score[static_cast<size_t>(l) * a.plane +
                         min(static_cast<int64_t>(chunk_begin(blockIdx.x) + tk), a.plane - 1)];
        __builtin_amdgcn_sched_barrier(0);  // every load is issued before the first wait
        if (!resolve_chunk<RAG>(a, blockIdx.x, it, c)) return;
    } else {
        if (!resolve_chunk<RAG>(a, blockIdx.x, it, c)) return;
        load(it.first, min(it.n_chunks, vz::kPairChunks), it.first + c);
    }
    const int nk = chunk_keys(c, it.len + 1);
    const int j = chunk_begin(c) + min(tk, nk - 1);
    float* const sc = a.score + static_cast<size_t>(l) * a.plane + it.base + j;
    if (!one || it.base != 0) ld.old = *sc;
    // (used only for tk < nk, where j is the slot the speculative load read)

    // the layer statistics and the chunk's factor of every head
#pragma unroll
    for (int u = 0; u < FINISH_ROUNDS; ++u) {
        if (16 * u >= Hq) break;
        const int h = 16 * u + t / 16;
        const float2 st =
            it.n_chunks <= vz::kPairChunks
                ? vz::merge_pairs(pr[u], it.n_chunks, t % 16, Exp2Weight())
                : vz::merge_all(part.ml + (static_cast<size_t>(l) * Hq + min(h, Hq - 1)) * a.nc_max + it.first,
                                it.n_chunks, t % 16, Exp2Weight());
        if (t % 16 == 0 && h < Hq) s_f[h] = Exp2Rel()(m_own[u], st.x) * (1.0f / st.y);
    }
    __syncthreads();
    const bool evict = !RAG && a.ev != 0;
    fold_finish(a, ld, s_f, sc, Hq, nk, j == it.len, evict);
    if constexpr (!RAG) {
        if (!evict) return;
        const vz_sel::EvictOne e{a.cnt, a.cnt_stride, a.ev_budget, a.ev_sink, a.ev_M};
        if (!vz_sel::last_of_layer(e, l, a.n_chunks)) return;
        const size_t row = static_cast<size_t>(l) * a.plane;
        const int Hkv = a.Hkv;
        vz_sel::evict_one_slot<OUT_THREADS, uint16_t, D>(e, a.score + row, a.pos + row, a.k_cache + row * Hkv * D,
                                                         a.v_cache + row * Hkv * D, static_cast<size_t>(a.plane) * D, Hkv,
                                                         a.len + 1, a.next_pos + 1);
    }
}

// Slots of a cache whose single eviction the folding launch does itself, where
// one block looks at every score of the layer (256 threads; 128 on the general
// path with several KV heads, whose sums its blocks also add up), against a
// launch of its own with 1024 threads per layer.  In a graph, folding launch
// and own launch, us:
//   chunked path        1,025 slots: 1 layer 9.1 and 11.4, 28 layers 18.7 and
//                       21.9; 8,193: 14.6 and 14.6, 16 layers 57.5 and 57.4,
//                       28 layers 107.1 and 106.6 (eager, one layer 15.2 and
//                       16.9: a launch less on the host)
//   general, 1 KV head  257: 10.8 and 13.5; 8,193: 19.0 and 19.9
//   2 and 4 KV heads    1,025: 14.0 and 16.3; 7,169: 20.5 and 20.9, 79.0 and
//                       80.1; 8,193: 22.4 and 21.8, 95.0 and 94.9
//   8                   5,121: 26.9 and 27.3, 84.6 and 85.6; 6,145: 27.7 and
//                       26.6, 99.0 and 98.6
//   16                  2,049: 48.1 and 48.9; 4,097: 202.6 and 201.6
//   32                  1,025: 32.0 and 34.2; 2,049: 55.2 and 53.5
// The chunked path takes it up to the whole-range path's length.
constexpr int64_t kEvictOneSlots = 8224;
int64_t evict_one_slots_general(int32_t Hkv) {
    return Hkv == 1 ? kEvictOneSlots : std::min<int64_t>(7168, 40960 / Hkv);
}

// Whether a call's outputs and scores are finished in one launch.  `chunks`:
// of a plane; `blocks`: fold and output blocks of a layer in that launch.
// One sequence: while its chunks' pairs are one round of loads (one layer 8.2
// against 10.1 us at 500 keys, 8.5 against 10.6 at 8000; 30 layers equal at
// 8000).  A batch: while its blocks are at most two rounds of the CUs' eight
// resident ones (4 x 2000 keys: one layer 9.1 against 11.4 us, 8 layers 30.9
// against 31.5, 16 layers 53.6 against 53.0, where the kernel's registers cost
// more than a launch), its sequences hold at most kPairChunks chunks on
// average, and its planes at most FINISH_BATCH_CHUNKS, which bounds what one
// sequence of nearly every slot costs (16 sequences of 1.2k-6.1k keys 26.9
// against 29.2 us; one of 80,000 keys, past the line, 45.8 against 40.6).
bool finish_in_one_launch(int64_t chunks, int seqs, int32_t L, int64_t blocks) {
    if (seqs == 1) return chunks <= vz::kPairChunks;
    return chunks <= std::min<int64_t>(FINISH_BATCH_CHUNKS, static_cast<int64_t>(vz::kPairChunks) * seqs) &&
           blocks * L <= FINISH_BATCH_BLOCKS;
}

template <int NW, bool RAG>
hipError_t launch_decode_fused(const VzDecodeArgs& v, hipStream_t stream) {
    FusedArgs a{};
    a.q = static_cast<const uint16_t*>(v.q);
    a.k_new = static_cast<const uint16_t*>(v.k_new);
    a.v_new = static_cast<const uint16_t*>(v.v_new);
    a.k_cache = static_cast<uint16_t*>(v.k_cache);
    a.v_cache = static_cast<uint16_t*>(v.v_cache);
    a.pos = v.pos;
    a.score = v.score;
    a.out = static_cast<uint16_t*>(v.out);
    a.ws = static_cast<uint8_t*>(v.ws);
    a.Hq = v.Hq;
    a.Hkv = NW;
    a.L = v.L;
    a.hdr_bytes = static_cast<int32_t>(vz_decode_hdr_bytes(v.L));
    a.scale_log2 = (v.sm_scale > 0.f ? v.sm_scale : 1.0f / sqrtf(static_cast<float>(D))) * kLog2e;
    a.gamma = v.gamma;
    a.rag = v.rag;
    int seqs = 1;
    if (RAG) {
        a.plane = v.rag.total;
        a.nc_max = static_cast<int32_t>(vz_decode_chunk_rows(a.plane, v.rag.n));
        a.n_chunks = a.nc_max;  // grid extent per layer
        seqs = v.rag.n;
    } else {
        a.plane = v.cap;
        a.len = v.len;
        a.next_pos = v.next_pos;
        a.n_chunks = static_cast<int32_t>((static_cast<int64_t>(v.len) + CHUNK) / CHUNK);  // of len + 1 keys
        a.nc_max = static_cast<int32_t>(vz_decode_chunk_rows(a.plane, 0));
    }
    if (!RAG) {
        a.cnt = vz_decode_counters(v.ws);
        a.tag = vz_call_tag();
        a.ev = v.ev;
        a.ev_budget = v.ev_budget;
        a.ev_sink = v.ev_sink;
        a.ev_M = v.ev_M;
        a.ev_kept = v.ev_kept;
        a.ev_n = v.ev_n;
    }
    if (vz_decode_range_ok(a.L, NW, RAG ? v.rag.n : 0)) {
        return vz_launch_decode_range(a, NW, stream);
    }
    if (a.ev) {  // counted in the finishing launch, which leaves the layer statistics' array (the last one) free
        const size_t end = vz_decode_fused_ws_bytes(a.L, a.Hq, a.plane, 0);
        a.cnt = reinterpret_cast<uint64_t*>(a.ws + end) - static_cast<size_t>(a.L) * a.Hq;
        a.cnt_stride = a.Hq;
    }
    hipLaunchKernelGGL((decode_attend_kernel<NW, RAG>), RAG ? dim3(a.n_chunks * NW, a.L) : dim3(a.L * a.n_chunks * NW),
                       dim3(64 * SPLIT_W), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (finish_in_one_launch((a.plane + CHUNK - 1) / CHUNK, seqs, a.L, a.n_chunks + a.Hq * static_cast<int64_t>(seqs))) {
        hipLaunchKernelGGL((decode_finish_kernel<RAG>), dim3(a.n_chunks + a.Hq * seqs, a.L), dim3(OUT_THREADS), 0,
                           stream, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((decode_output_kernel<RAG>), dim3(a.Hq, a.L, seqs), dim3(OUT_THREADS), 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_fold_kernel<RAG>), dim3(a.n_chunks, a.L), dim3(OUT_THREADS), 0, stream, a);
    return hipGetLastError();
}

template <int NW>
hipError_t launch_decode_fused_any(const VzDecodeArgs& v, hipStream_t stream) {
    return v.rag.n > 0 ? launch_decode_fused<NW, true>(v, stream) : launch_decode_fused<NW, false>(v, stream);
}

}  // namespace

// ---- sizing shared with the host API ----
// Chunk rows of the partials per layer: ceil(plane / CHUNK) for a single
// sequence; for a ragged call ceil(plane / CHUNK) + n_seqs, a bound on the
// sum of ceil((len[s] + 1) / CHUNK) over sequences that lie inside the planes
// without overlapping.
int64_t vz_decode_chunk_rows(int64_t plane, int32_t n_seqs) {
    return (plane + CHUNK - 1) / CHUNK + (n_seqs > 0 ? n_seqs : 0);
}

size_t vz_decode_hdr_bytes(int32_t L) {
    return kHeaderBytes + (static_cast<size_t>(L) * sizeof(uint64_t) + 255) / 256 * 256;
}

uint64_t* vz_decode_counters(void* ws) {
    return reinterpret_cast<uint64_t*>(static_cast<uint8_t*>(ws) + kHeaderBytes);
}

uint32_t vz_call_tag() {
    static std::atomic<uint32_t> next{static_cast<uint32_t>(std::random_device{}())};
    uint32_t t;
    do t = next.fetch_add(1, std::memory_order_relaxed);
    while (t == 0);
    return t;
}

bool vz_decode_fused_ok(int32_t dtype, int32_t d, int32_t Hq, int32_t Hkv, int32_t L, int64_t plane, int32_t n_seqs) {
    if (dtype != VZ_BF16 || d != D) return false;
    if (!(Hkv == 1 || Hkv == 2 || Hkv == 4 || Hkv == 8)) return false;
    if (Hq % Hkv != 0 || Hq / Hkv > GMAX) return false;
    // 32-bit chunk-row indexes of the partials (the attend grid is smaller)
    return static_cast<int64_t>(L) * vz_decode_chunk_rows(plane, n_seqs) * Hq < (int64_t(1) << 31);
}

size_t vz_decode_fused_ws_bytes(int32_t L, int32_t Hq, int64_t plane, int32_t n_seqs) {
    const int64_t rows = vz_decode_chunk_rows(plane, n_seqs);
    const int32_t seqs = n_seqs > 0 ? n_seqs : 1;
    return vz_decode_hdr_bytes(L) + static_cast<size_t>(L) * rows * Hq * (sizeof(float2) + sizeof(uint16_t) * (D + CHUNK)) +
           static_cast<size_t>(seqs) * L * Hq * sizeof(float2);
}

hipError_t vz_launch_decode_fused(const VzDecodeArgs& a, hipStream_t stream) {
    switch (a.Hkv) {
        case 1: return launch_decode_fused_any<1>(a, stream);
        case 2: return launch_decode_fused_any<2>(a, stream);
        case 4: return launch_decode_fused_any<4>(a, stream);
        case 8: return launch_decode_fused_any<8>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

bool vz_decode_takes_range(const VzDecodeArgs& a) {
    return a.rag.n == 0 && vz_decode_fused_ok(a.dtype, a.d, a.Hq, a.Hkv, a.L, a.cap, 0) &&
           vz_decode_range_ok(a.L, a.Hkv, 0) && vz_decode_range_whole(a.len);
}

bool vz_decode_evicts(const VzDecodeArgs& a, int32_t budget, bool kept) {
    const int64_t T = static_cast<int64_t>(a.len) + 1;
    const int64_t E = T > budget ? T - budget : 0;
    if (vz_decode_takes_range(a)) return a.Hkv <= 4 && E <= vz_sel::kInlineRows;
    if (E != 1 || kept || T > kEvictOneSlots) return false;
    if (!vz_decode_fused_ok(a.dtype, a.d, a.Hq, a.Hkv, a.L, a.cap, 0)) return T <= evict_one_slots_general(a.Hkv);
    return !vz_decode_range_ok(a.L, a.Hkv, 0) &&
           finish_in_one_launch((static_cast<int64_t>(a.cap) + CHUNK - 1) / CHUNK, 1, a.L, 0);
}
