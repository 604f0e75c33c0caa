// Stage-1 semantic-anchored fusion (Sec. 3.2.1, Eq. 4 group means plus the
// additive anchor, Eq. 5 order) as a segmented mean over K/V rows.
// Head sizes 64 and 128 (K/V-space fusion) use the lane-group kernel below;
// wider rows -- the embedding-space form, one "head" of width d_model -- use
// a kernel with one block per span that sweeps the row in 16-byte columns.
// Either kernel fuses K and V, or K alone when no V is given.
//
// Work split: a "lane group" of D/ (16 bytes / element size) lanes owns one
// (layer, KV head, K-or-V, span); each lane owns 16 contiguous bytes of the
// row, so a group reads whole rows with 16-byte loads and a wave streams
// 64 * 16 = 1 KB per load instruction.  Rows of a span are contiguous in HBM;
// the loop keeps four rows in flight per lane.  Accumulation is float32 in row
// order; the mean is an IEEE division by the span length, so a length-1 span
// reproduces its row bit for bit.
#include <algorithm>
#include <type_traits>

#include "vz_internal.h"

namespace {

struct FuseArgs {
    const void* k_in;
    const void* v_in;
    const int32_t* off;
    const void* ak;
    const void* av;
    void* k_out;
    void* v_out;
    float* score_out;
    int32_t* pos_out;
    int32_t H;
    int32_t kinds;              // 2: K and V, 1: K only
    int32_t d;                  // row length (the wide-row kernel)
    int32_t T_in, n_spans;      // single sequence
    int64_t in_plane, out_plane;  // rows per (layer, head) plane of the input and of the output
    int32_t blocks_per_seq;     // ragged: span blocks per sequence in grid x
    // ragged batch (n_seqs > 0): sequence s reads input rows in_base[s] ..
    // + T_in[s] and offsets off[off_base[s] .. + n_spans[s]], writes output
    // slots base[s] .. + n_spans[s] (cap[s] slots are its own)
    int32_t n_seqs;
    const int64_t* in_base;
    const int32_t* T_in_s;
    const int64_t* off_base;
    const int32_t* n_spans_s;
    const int64_t* base;
    const int32_t* cap;
    int32_t* status;
    int64_t total_off;
    int32_t max_spans;
};

// Status of sequence s of a ragged fusion (VZ_OK when it can be served,
// VZ_IDLE for an idle slot).
__device__ int ragged_fuse_status(const FuseArgs& a, int s) {
    const int64_t ib = a.in_base[s], ob = a.off_base[s], b = a.base[s];
    const int T = a.T_in_s[s], n = a.n_spans_s[s], c = a.cap[s];
    if (c == 0) return VZ_IDLE;
    if (T < 0 || n < 0 || c < 1 || ib < 0 || ib > a.in_plane - T || ob < 0 || ob > a.total_off - n - 1 || b < 0 ||
        b > a.out_plane - c)
        return VZ_ERR_INVALID;
    if (n > T) return VZ_ERR_SHAPE;
    if (n > c || n > a.max_spans) return VZ_ERR_CAPACITY;
    return VZ_OK;
}

// Adds rows [b, e) of NC 16-byte columns (gap elements apart) to acc in row
// order (col: row 0 of the first, stride elements per row), four rows' loads
// at a time.  bfloat16: the loads of the remainder go out together too, those
// past the span reading its last row again (a cache hit) and adding nothing, so
// no row waits for another's round trip; a remainder of up to three rows, one
// load after the other, is most of a span of mean length 4 (12 layers x 4 heads
// x 32,768 rows: mean length 1.2: 305 -> 304 us, 1.5: 277 -> 260, 2: 242 ->
// 224, 3: 196 -> 185, 5: 176 -> 177, 8: 186 -> 186, 12: 175 -> 175; every round
// masked, full ones too, costs 4 % at 1.2 and 1 % at 8 and 12; 48 layers, mean
// length 4.02: 706-724 either way, by where the buffers lie).  Two columns per
// thread: every round masked in one loop (3584 elements, mean length 4.02: 74.9
// -> 69.2 us, 70.2 with the remainder by itself).  float32 rows are twice as
// long and the repeated reads cost what they save (222 against 227 us at 12
// layers x 20,000 rows): the remainder goes row by row.
template <int DT, int NC>
__device__ __forceinline__ void add_rows(const typename vz::Elem<DT>::T* col, size_t stride, int gap, int32_t b,
                                         int32_t e, float (*acc)[vz::Elem<DT>::kPer16B]) {
    constexpr int PER = vz::Elem<DT>::kPer16B, ROWS = 4;
    constexpr bool MASKED = DT == VZ_BF16, ONE_LOOP = MASKED && NC > 1;
    auto add = [&](const uint4 (&x)[NC], bool on) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            float f[PER];
            vz::unpack16<DT>(x[c], f);
#pragma unroll
            for (int i = 0; i < PER; ++i) acc[c][i] += on ? f[i] : 0.f;
        }
    };
    auto load = [&](int32_t r, uint4 (&x)[NC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            x[c] = *reinterpret_cast<const uint4*>(col + static_cast<size_t>(r) * stride + c * gap);
    };
    int32_t r = b;
    for (; ONE_LOOP ? r < e : r + ROWS <= e; r += ROWS) {
        uint4 x[ROWS][NC];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) load(ONE_LOOP ? min(r + u, e - 1) : r + u, x[u]);
#pragma unroll
        for (int u = 0; u < ROWS; ++u) add(x[u], !ONE_LOOP || r + u < e);
    }
    if constexpr (MASKED && !ONE_LOOP) {
        if (r < e) {
            uint4 x[ROWS - 1][NC];
#pragma unroll
            for (int u = 0; u < ROWS - 1; ++u) load(min(r + u, e - 1), x[u]);
#pragma unroll
            for (int u = 0; u < ROWS - 1; ++u) add(x[u], r + u < e);
        }
    } else if constexpr (!MASKED) {
        for (; r < e; ++r) {
            uint4 x[NC];
            load(r, x);
            add(x, true);
        }
    }
}

template <int DT, int D, bool RAG>
__global__ __launch_bounds__(256) void fuse_spans_kernel(const FuseArgs a) {
    using E = vz::Elem<DT>;
    using T = typename E::T;
    constexpr int PER = E::kPer16B;      // elements per 16-byte vector
    constexpr int LANES = D / PER;       // lanes per span row
    constexpr int SPB = 256 / LANES;     // spans per block

    const int sub = threadIdx.x / LANES;
    const int lane = threadIdx.x % LANES;
    const int which = blockIdx.y % a.kinds;  // 0: K, 1: V
    const int h = blockIdx.y / a.kinds;
    const int l = blockIdx.z;
    int bx = blockIdx.x, T_in = a.T_in, n_spans = a.n_spans;
    int64_t in_row = 0, out_row = 0;  // first row of the sequence in its planes
    const int32_t* off = a.off;
    if constexpr (RAG) {
        const int s = blockIdx.x / a.blocks_per_seq;
        bx = blockIdx.x - s * a.blocks_per_seq;
        const int st = ragged_fuse_status(a, s);
        if (a.status && bx == 0 && blockIdx.y == 0 && l == 0 && threadIdx.x == 0) a.status[s] = st;
        if (st != VZ_OK) return;
        T_in = a.T_in_s[s];
        n_spans = a.n_spans_s[s];
        in_row = a.in_base[s];
        out_row = a.base[s];
        off = a.off + a.off_base[s];
    }
    const int64_t j = static_cast<int64_t>(bx) * SPB + sub;
    if (j >= n_spans) return;

    int32_t b = off[j], e = off[j + 1];
    b = b < 0 ? 0 : (b > T_in ? T_in : b);
    e = e < b ? b : (e > T_in ? T_in : e);

    const T* src = static_cast<const T*>(which ? a.v_in : a.k_in) +
                   ((static_cast<size_t>(l) * a.H + h) * static_cast<size_t>(a.in_plane) + in_row) * D + lane * PER;
    float sum[1][PER];
    float* const acc = sum[0];
#pragma unroll
    for (int i = 0; i < PER; ++i) acc[i] = 0.f;
    add_rows<DT, 1>(src, D, 0, b, e, sum);
    const float cnt = static_cast<float>(e - b);
#pragma unroll
    for (int i = 0; i < PER; ++i) acc[i] = (e > b) ? acc[i] / cnt : 0.f;

    const T* anchor = static_cast<const T*>(which ? a.av : a.ak);
    const size_t orow = (static_cast<size_t>(l) * a.H + h) * static_cast<size_t>(a.out_plane) + out_row + j;
    if (anchor) {
        // single sequence: [L][H][n_spans][d]; ragged: laid out like the output
        const size_t arow = RAG ? orow : (static_cast<size_t>(l) * a.H + h) * static_cast<size_t>(n_spans) + j;
        uint4 x = *reinterpret_cast<const uint4*>(anchor + arow * D + lane * PER);
        float f[PER];
        vz::unpack16<DT>(x, f);
#pragma unroll
        for (int i = 0; i < PER; ++i) acc[i] += f[i];
    }
    T* dst = static_cast<T*>(which ? a.v_out : a.k_out) + orow * D + lane * PER;
    *reinterpret_cast<uint4*>(dst) = vz::pack16<DT>(acc);

    if (which == 0 && h == 0 && lane == 0) {
        const size_t prow = static_cast<size_t>(l) * a.out_plane + out_row + j;
        a.pos_out[prow] = static_cast<int32_t>(j);
        a.score_out[prow] = 0.f;
    }
}

// Wide rows (d a multiple of one 16-byte vector, other than 64 and 128): one
// block per (span, K-or-V, head, layer); thread t owns the 16-byte columns t,
// t + threads, ... of the row, NC of them at a time, and sums them over the
// span's rows in row order, as the lane-group kernel does, so the arithmetic
// is the same.  Two columns at a time (two_columns) keep eight loads in flight
// per thread instead of one to four, at 81 registers and five waves per SIMD
// instead of 41 and eight; rows of up to WIDE_THREADS columns take a block of
// as many waves as they need.
constexpr int WIDE_THREADS = 256;
template <int DT, bool RAG, int NC>
__global__ __launch_bounds__(WIDE_THREADS) void fuse_wide_kernel(const FuseArgs a) {
    using E = vz::Elem<DT>;
    using T = typename E::T;
    constexpr int PER = E::kPer16B;
    const int nv = a.d / PER;  // 16-byte columns per row
    const int which = blockIdx.y % a.kinds;
    const int h = blockIdx.y / a.kinds;
    const int l = blockIdx.z;
    int64_t j = blockIdx.x;
    int T_in = a.T_in, n_spans = a.n_spans;
    int64_t in_row = 0, out_row = 0;
    const int32_t* off = a.off;
    if constexpr (RAG) {
        const int s = static_cast<int>(blockIdx.x / a.blocks_per_seq);
        j = blockIdx.x - static_cast<int64_t>(s) * a.blocks_per_seq;
        const int st = ragged_fuse_status(a, s);
        if (a.status && j == 0 && blockIdx.y == 0 && l == 0 && threadIdx.x == 0) a.status[s] = st;
        if (st != VZ_OK) return;
        T_in = a.T_in_s[s];
        n_spans = a.n_spans_s[s];
        in_row = a.in_base[s];
        out_row = a.base[s];
        off = a.off + a.off_base[s];
    }
    if (j >= n_spans) return;
    int32_t b = off[j], e = off[j + 1];
    b = b < 0 ? 0 : (b > T_in ? T_in : b);
    e = e < b ? b : (e > T_in ? T_in : e);
    const float cnt = static_cast<float>(e - b);
    const T* src = static_cast<const T*>(which ? a.v_in : a.k_in) +
                   ((static_cast<size_t>(l) * a.H + h) * static_cast<size_t>(a.in_plane) + in_row) * a.d;
    const T* anchor = static_cast<const T*>(which ? a.av : a.ak);
    const size_t orow = (static_cast<size_t>(l) * a.H + h) * static_cast<size_t>(a.out_plane) + out_row + j;
    const size_t arow = RAG ? orow : (static_cast<size_t>(l) * a.H + h) * static_cast<size_t>(n_spans) + j;
    T* dst = static_cast<T*>(which ? a.v_out : a.k_out) + orow * a.d;
    const int threads = blockDim.x;
    auto columns = [&](auto n, int c0) {
        constexpr int N = decltype(n)::value;
        float acc[N][PER];
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
            for (int i = 0; i < PER; ++i) acc[k][i] = 0.f;
        add_rows<DT, N>(src + c0 * PER, a.d, WIDE_THREADS * PER, b, e, acc);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int c = c0 + k * WIDE_THREADS;
#pragma unroll
            for (int i = 0; i < PER; ++i) acc[k][i] = (e > b) ? acc[k][i] / cnt : 0.f;
            if (anchor) {
                const uint4 x = *reinterpret_cast<const uint4*>(anchor + arow * a.d + c * PER);
                float f[PER];
                vz::unpack16<DT>(x, f);
#pragma unroll
                for (int i = 0; i < PER; ++i) acc[k][i] += f[i];
            }
            *reinterpret_cast<uint4*>(dst + c * PER) = vz::pack16<DT>(acc[k]);
        }
    };
    for (int c = threadIdx.x; c < nv; c += NC * threads) {
        // whole waves take NC columns: a wave whose lanes differ would run both forms
        const int last = __builtin_amdgcn_readfirstlane((c | (vz::kWave - 1)) + (NC - 1) * WIDE_THREADS);
        if (NC > 1 && last < nv) columns(std::integral_constant<int, NC>{}, c);
        else for (int k = c; k < min(nv, c + NC * threads); k += threads) columns(std::integral_constant<int, 1>{}, k);
    }
    if (which == 0 && h == 0 && threadIdx.x == 0) {
        const size_t prow = static_cast<size_t>(l) * a.out_plane + out_row + j;
        a.pos_out[prow] = static_cast<int32_t>(j);
        a.score_out[prow] = 0.f;
    }
}

template <int DT, int NC>
hipError_t launch_wide(const FuseArgs& a, int32_t L, hipStream_t stream) {
    const int nv = a.d / vz::Elem<DT>::kPer16B;
    const dim3 block(std::min(WIDE_THREADS, (nv + vz::kWave - 1) / vz::kWave * vz::kWave));
    if (a.n_seqs > 0) {
        FuseArgs r = a;
        r.blocks_per_seq = a.max_spans > 0 ? a.max_spans : 1;  // still report every sequence's status
        dim3 grid(static_cast<unsigned>(static_cast<int64_t>(r.blocks_per_seq) * a.n_seqs), a.kinds * a.H, L);
        hipLaunchKernelGGL((fuse_wide_kernel<DT, true, NC>), grid, block, 0, stream, r);
        return hipGetLastError();
    }
    if (a.n_spans == 0) return hipSuccess;
    dim3 grid(a.n_spans, a.kinds * a.H, L);
    hipLaunchKernelGGL((fuse_wide_kernel<DT, false, NC>), grid, block, 0, stream, a);
    return hipGetLastError();
}
// Whether rows of nv columns in spans of mean length rows / spans take two
// columns per thread.  32,768 rows of 3584 elements or as many bytes of others,
// one and two columns, us: 8192 elements, mean length 1.0: 81.5 and 82.5, 1.2:
// 73.0 and 71.9, 4.02: 56.1 and 53.6; 5120, 1.2: 70.8 and 75.5, 2.0: 57.2 and
// 55.0; 3584, 1.0: 76.0 and 86.6, 1.5: 61.3 and 62.3, 1.75: 91.3 and 88.7 (all
// 32,768 rows), 4.02: 47.9 and 44.6; 2560, 2.0: 54.6 and 56.3, 4.02: 48.9 and
// 44.9.  Below 320 columns no wave has two.  float32 (remainders row by row)
// gains a little or nothing at every mean length: 2048 elements, 1.0: 86.8 and
// 86.1, 8.0: 50.9 and 49.0.  (A ragged call's spans are bounded by max_spans
// per sequence.)
template <int DT>
bool two_columns(int32_t nv, int64_t rows, int64_t spans) {
    if (nv < WIDE_THREADS + vz::kWave) return false;
    if (DT == VZ_F32) return true;
    if (nv >= 768) return 5 * rows >= 6 * spans;
    return nv >= 448 ? 4 * rows >= 7 * spans : rows >= 3 * spans;
}
template <int DT>
hipError_t launch_wide_any(const FuseArgs& a, int32_t L, hipStream_t stream) {
    const int64_t rows = a.n_seqs > 0 ? a.in_plane : a.T_in;
    const int64_t spans = a.n_seqs > 0 ? static_cast<int64_t>(a.max_spans) * a.n_seqs : a.n_spans;
    return two_columns<DT>(a.d / vz::Elem<DT>::kPer16B, rows, spans) ? launch_wide<DT, 2>(a, L, stream)
                                                                    : launch_wide<DT, 1>(a, L, stream);
}

template <int DT, int D>
hipError_t launch(const FuseArgs& a, int32_t L, hipStream_t stream) {
    constexpr int SPB = 256 / (D / vz::Elem<DT>::kPer16B);
    if (a.n_seqs > 0) {
        FuseArgs r = a;
        r.blocks_per_seq = (a.max_spans + SPB - 1) / SPB;
        if (r.blocks_per_seq == 0) r.blocks_per_seq = 1;  // still report every sequence's status
        dim3 grid(static_cast<unsigned>(static_cast<int64_t>(r.blocks_per_seq) * a.n_seqs), a.kinds * a.H, L);
        hipLaunchKernelGGL((fuse_spans_kernel<DT, D, true>), grid, dim3(256), 0, stream, r);
        return hipGetLastError();
    }
    if (a.n_spans == 0) return hipSuccess;
    dim3 grid((a.n_spans + SPB - 1) / SPB, a.kinds * a.H, L);
    hipLaunchKernelGGL((fuse_spans_kernel<DT, D, false>), grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t dispatch(FuseArgs a, int32_t L, int32_t d, int32_t dtype, hipStream_t stream) {
    a.kinds = a.v_in ? 2 : 1;
    a.d = d;
    if (dtype == VZ_BF16 && d == 128) return launch<VZ_BF16, 128>(a, L, stream);
    if (dtype == VZ_BF16 && d == 64) return launch<VZ_BF16, 64>(a, L, stream);
    if (dtype == VZ_F32 && d == 128) return launch<VZ_F32, 128>(a, L, stream);
    if (dtype == VZ_F32 && d == 64) return launch<VZ_F32, 64>(a, L, stream);
    if (dtype == VZ_BF16 && d % vz::Elem<VZ_BF16>::kPer16B == 0) return launch_wide_any<VZ_BF16>(a, L, stream);
    if (dtype == VZ_F32 && d % vz::Elem<VZ_F32>::kPer16B == 0) return launch_wide_any<VZ_F32>(a, L, stream);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t vz_launch_fuse(const void* k_in, const void* v_in, int32_t T_in, const int32_t* off,
                          int32_t n_spans, const void* ak, const void* av, void* k_out, void* v_out,
                          float* score_out, int32_t* pos_out, int32_t L, int32_t H, int32_t d,
                          int32_t cap_out, int32_t dtype, hipStream_t stream) {
    FuseArgs a{};
    a.k_in = k_in;
    a.v_in = v_in;
    a.off = off;
    a.ak = ak;
    a.av = av;
    a.k_out = k_out;
    a.v_out = v_out;
    a.score_out = score_out;
    a.pos_out = pos_out;
    a.H = H;
    a.T_in = T_in;
    a.n_spans = n_spans;
    a.in_plane = T_in;
    a.out_plane = cap_out;
    return dispatch(a, L, d, dtype, stream);
}

hipError_t vz_launch_fuse_ragged(const VzFuseRaggedArgs& g, hipStream_t stream) {
    FuseArgs a{};
    a.k_in = g.k_in;
    a.v_in = g.v_in;
    a.off = g.span_off;
    a.ak = g.anchor_k;
    a.av = g.anchor_v;
    a.k_out = g.k_out;
    a.v_out = g.v_out;
    a.score_out = g.score_out;
    a.pos_out = g.pos_out;
    a.H = g.Hkv;
    a.in_plane = g.total_in;
    a.out_plane = g.total;
    a.n_seqs = g.n_seqs;
    a.in_base = g.in_base;
    a.T_in_s = g.T_in;
    a.off_base = g.off_base;
    a.n_spans_s = g.n_spans;
    a.base = g.seq_base;
    a.cap = g.cap;
    a.status = g.status;
    a.total_off = g.total_off;
    a.max_spans = g.max_spans;
    return dispatch(a, g.L, g.d, g.dtype, stream);
}
