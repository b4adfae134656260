// Convolution layers with CSR filter banks, computed directly on the
// batch-contiguous maps (no lowered operand for the products):
//
//   forward     Y[(co,oh,ow)][b] = sum_{p in row co} w_p X[(ci, oh*SH-PH+kh, ow*SW-PW+kw)][b]
//   backward    dX[(ci,ih,iw)][b] = sum over CSC entries q of the columns (ci,kh,kw)
//               with ih = oh*SH-PH+kh, iw = ow*SW-PW+kw of w_q dY[(co_q,oh,ow)][b]
//   im2col      the lowered operand Xcol[(ci,kh,kw)][(oh*OW+ow)*B + b], used only
//               for the weight gradient (a dense contraction: matrix cores, or
//               the pattern-sampled product)
//   max pool    Y[(c,oh,ow)][b] = max of the KH x KW window
//
// A filter column is (ci*KH + kh)*KW + kw (Caffe's im2col row order).  Each
// output is summed by one thread in a fixed order (forward: CSR order;
// backward: kh, kw, then CSC order), so results are reproducible.  The input
// maps of LeNet-sized layers fit in L2, so the shifted re-reads of X by the
// direct products stay on chip; only the lowered operand of the weight
// gradient is streamed from HBM.
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace l1csr {

namespace {

constexpr int kThreads = 256;
constexpr int kStage = 2048;  // filter entries staged in LDS per pass
constexpr int kBatch = 8;     // entries whose loads are in flight together
constexpr int kMaxKK = 1024;  // filter positions KH*KW per channel (backward)

struct geom_t {
    int C, H, W, KH, KW, SH, SW, PH, PW, OH, OW;
};

geom_t to_geom(const conv_geom &g) {
    geom_t t;
    t.C = g.C; t.H = g.H; t.W = g.W; t.KH = g.KH; t.KW = g.KW;
    t.SH = g.SH; t.SW = g.SW; t.PH = g.PH; t.PW = g.PW;
    t.OH = (g.H + 2 * g.PH - g.KH) / g.SH + 1;
    t.OW = (g.W + 2 * g.PW - g.KW) / g.SW + 1;
    return t;
}

template <int VEC>
struct vec_t;
template <>
struct vec_t<1> {
    typedef float T;
    static __device__ __forceinline__ T load(const float *p) { return *p; }
    static __device__ __forceinline__ void store(float *p, T v) { *p = v; }
    static __device__ __forceinline__ void fma(T &a, float w, T x) { a = fmaf(w, x, a); }
    static __device__ __forceinline__ T zero() { return 0.f; }
    static __device__ __forceinline__ void vmax(T &a, T x) { a = x > a ? x : a; }
};
template <>
struct vec_t<2> {
    typedef float2 T;
    static __device__ __forceinline__ T load(const float *p) { return *reinterpret_cast<const float2 *>(p); }
    static __device__ __forceinline__ void store(float *p, T v) { *reinterpret_cast<float2 *>(p) = v; }
    static __device__ __forceinline__ void fma(T &a, float w, T x) {
        a.x = fmaf(w, x.x, a.x);
        a.y = fmaf(w, x.y, a.y);
    }
    static __device__ __forceinline__ T zero() { return make_float2(0.f, 0.f); }
};
template <>
struct vec_t<4> {
    typedef float4 T;
    static __device__ __forceinline__ T load(const float *p) { return *reinterpret_cast<const float4 *>(p); }
    static __device__ __forceinline__ void store(float *p, T v) { *reinterpret_cast<float4 *>(p) = v; }
    static __device__ __forceinline__ void fma(T &a, float w, T x) {
        a.x = fmaf(w, x.x, a.x);
        a.y = fmaf(w, x.y, a.y);
        a.z = fmaf(w, x.z, a.z);
        a.w = fmaf(w, x.w, a.w);
    }
    static __device__ __forceinline__ T zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
    static __device__ __forceinline__ void vmax(T &a, T x) {
        a.x = x.x > a.x ? x.x : a.x;
        a.y = x.y > a.y ? x.y : a.y;
        a.z = x.z > a.z ? x.z : a.z;
        a.w = x.w > a.w ? x.w : a.w;
    }
};

// Forward.  Block (co, slice): the output block of channel co is the flattened
// [OH*OW][B] range f = pos*B + b; each thread takes VEC consecutive f of one
// position (B % VEC == 0).  Row co's entries are decoded into LDS once per
// pass: the input-row offset of output position (0, 0) and (kh, kw) for the
// range test.
template <int VEC>
__global__ __launch_bounds__(kThreads) void conv_fwd_kernel(geom_t g, int B, const int *__restrict__ ptr,
                                                            const int *__restrict__ idx,
                                                            const float *__restrict__ vals,
                                                            const float *__restrict__ X, int64_t ldx,
                                                            float *__restrict__ Y, int64_t ldy, int slices) {
    typedef vec_t<VEC> V;
    __shared__ int off_s[kStage];
    __shared__ int khw_s[kStage];
    __shared__ float w_s[kStage];
    const int co = blockIdx.x;
    const int64_t F = (int64_t)g.OH * g.OW * B;
    const int s = ptr[co], e = ptr[co + 1];
    auto stage = [&](int p0, int n) {
        __syncthreads();  // the previous entries are consumed
        for (int i = threadIdx.x; i < n; i += kThreads) {
            const int col = idx[p0 + i];
            const int ci = col / (g.KH * g.KW);
            const int r = col - ci * g.KH * g.KW;
            const int kh = r / g.KW, kw = r - kh * g.KW;
            off_s[i] = (ci * g.H + kh) * g.W + kw;
            khw_s[i] = (kh << 16) | kw;
            w_s[i] = vals[p0 + i];
        }
        __syncthreads();
    };
    const bool one_pass = e - s <= kStage;
    if (one_pass) stage(s, e - s);  // once for every slice of this block
    // the block walks slices blockIdx.y, blockIdx.y + gridDim.y, ... of channel co
    for (int slice = blockIdx.y; slice < slices; slice += gridDim.y) {
        const int64_t f = ((int64_t)slice * kThreads + threadIdx.x) * VEC;
        const bool active = f < F;
        const int pos = active ? (int)(f / B) : 0;
        const int b = active ? (int)(f - (int64_t)pos * B) : 0;
        const int oh = pos / g.OW, ow = pos - oh * g.OW;
        const int ih0 = oh * g.SH - g.PH, iw0 = ow * g.SW - g.PW;
        const int64_t base = (int64_t)(ih0 * g.W + iw0);
        typename V::T acc = V::zero();
        for (int p0 = s; p0 < e; p0 += kStage) {
            const int n = min(kStage, e - p0);
            if (!one_pass) stage(p0, n);
            if (!active) continue;
            // kBatch entries' loads in flight at a time; an entry whose input
            // position is outside the map loads row 0 instead and is skipped
            for (int i0 = 0; i0 < n; i0 += kBatch) {
                typename V::T x[kBatch];
                bool ok[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int i = i0 + u < n ? i0 + u : n - 1;
                    const int kh = khw_s[i] >> 16, kw = khw_s[i] & 0xffff;
                    const int ih = ih0 + kh, iw = iw0 + kw;
                    ok[u] = i0 + u < n && ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
                    x[u] = V::load(X + (ok[u] ? (base + off_s[i]) * ldx : 0) + b);
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u)
                    if (ok[u]) V::fma(acc, w_s[i0 + u], x[u]);
            }
        }
        if (active) V::store(Y + ((int64_t)co * g.OH * g.OW + pos) * ldy + b, acc);
    }
}

// Backward for the input maps.  Block (ci, slice) over the flattened
// [H*W][B] range of channel ci; the CSC columns (ci, kh, kw), kh, kw in order,
// are staged as (output-channel row offset, kh, kw, value).
template <int VEC>
__global__ __launch_bounds__(kThreads) void conv_bwd_kernel(geom_t g, int B, const int *__restrict__ col_ptr,
                                                            const int *__restrict__ row_idx,
                                                            const float *__restrict__ vals_t,
                                                            const float *__restrict__ dY, int64_t ldy,
                                                            float *__restrict__ dX, int64_t ldx, int slices) {
    typedef vec_t<VEC> V;
    __shared__ int co_s[kStage];
    __shared__ int khw_s[kStage];
    __shared__ float w_s[kStage];
    __shared__ int cp_s[kMaxKK + 1];
    const int ci = blockIdx.x;
    const int64_t F = (int64_t)g.H * g.W * B;
    const int kk = g.KH * g.KW;
    // the column pointers of this channel's KH*KW filter columns (kk <= kMaxKK)
    for (int c = threadIdx.x; c <= kk; c += kThreads) cp_s[c] = col_ptr[ci * kk + c];
    __syncthreads();
    const int s = cp_s[0], e = cp_s[kk];
    auto stage = [&](int q0, int n) {
        __syncthreads();
        for (int i = threadIdx.x; i < n; i += kThreads) {
            // the filter column of CSC entry q0 + i: last c with cp_s[c] <= q0 + i
            const int q = q0 + i;
            int lo = 0, hi = kk - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (cp_s[mid] <= q) lo = mid; else hi = mid - 1;
            }
            const int kh = lo / g.KW, kw = lo - kh * g.KW;
            co_s[i] = row_idx[q];
            khw_s[i] = (kh << 16) | kw;
            w_s[i] = vals_t[q];
        }
        __syncthreads();
    };
    const bool one_pass = e - s <= kStage;
    if (one_pass) stage(s, e - s);
    for (int slice = blockIdx.y; slice < slices; slice += gridDim.y) {
        const int64_t f = ((int64_t)slice * kThreads + threadIdx.x) * VEC;
        const bool active = f < F;
        const int pos = active ? (int)(f / B) : 0;
        const int b = active ? (int)(f - (int64_t)pos * B) : 0;
        const int ih = pos / g.W, iw = pos - ih * g.W;
        typename V::T acc = V::zero();
        for (int q0 = s; q0 < e; q0 += kStage) {
            const int n = min(kStage, e - q0);
            if (!one_pass) stage(q0, n);
            if (!active) continue;
            for (int i0 = 0; i0 < n; i0 += kBatch) {
                typename V::T y[kBatch];
                bool ok[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int i = i0 + u < n ? i0 + u : n - 1;
                    const int kh = khw_s[i] >> 16, kw = khw_s[i] & 0xffff;
                    const int th = ih + g.PH - kh, tw = iw + g.PW - kw;  // oh*SH, ow*SW
                    const int oh = th >= 0 ? th / g.SH : -1, ow = tw >= 0 ? tw / g.SW : -1;
                    ok[u] = i0 + u < n && oh >= 0 && ow >= 0 && oh * g.SH == th && ow * g.SW == tw &&
                            oh < g.OH && ow < g.OW;
                    const int64_t row = ok[u] ? (int64_t)(co_s[i] * g.OH + oh) * g.OW + ow : 0;
                    y[u] = V::load(dY + row * ldy + b);
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u)
                    if (ok[u]) V::fma(acc, w_s[i0 + u], y[u]);
            }
        }
        if (active) V::store(dX + ((int64_t)ci * g.H * g.W + pos) * ldx + b, acc);
    }
}

constexpr int wave_positions(bool bwd) { return bwd ? 1 : 2; }

// Both products for batches that fill a wave's lanes: a wave takes PB
// consecutive output positions of a channel and 64 * VEC batch columns, so an
// entry's input row is the same for the whole wave.  The index arithmetic runs
// with an entry per lane, 64 at a time (the thread-per-output kernels above
// repeat it in every thread, 4 divisions an entry in the backward one), and a
// ballot drops the entries that fall outside the map; the rows and values of
// the others are then read from their lanes as scalars, and the loads of NB
// entries at PB positions are in flight together (an entry outside the map for
// one of the positions loads row 0 and is skipped).  Entries are summed in the order of
// the kernels above, so the bits are theirs.  Bound by the gathers through L1 and
// L2 (1 KB per entry and position) and, where a channel has few entries, by the
// stores.  conv2 of LeNet-5 at batch 256, thread-per-output -> this kernel: 17.7
// -> 12.8 us forward, 56.6 -> 15.8 backward; at 1024 33.2 -> 27.6 and 117 -> 47; its
// conv1 forward at 1024 34.7 -> 22.8.  Two positions and four entries a time
// forward, one and eight backward (its neighbours' valid entries differ): conv1
// forward with one and eight 30.1, conv2 backward with two and eight 21.8.
template <int VEC, bool BWD, bool MAPPED>
__global__ __launch_bounds__(kThreads) void conv_wave_kernel(geom_t g, int B, int chunks,
                                                             const int *__restrict__ ptr,
                                                             const int *__restrict__ idx,
                                                             const float *__restrict__ vals,
                                                             const float *__restrict__ in, int64_t ldi,
                                                             float *__restrict__ out, int64_t ldo, int tasks, int slices) {
    typedef vec_t<VEC> V;
    constexpr int kPB = wave_positions(BWD), kNB = BWD ? 8 : 4;
    __shared__ int map_s[kStage];  // first row of the entry's input map
    __shared__ int khw_s[kStage];
    __shared__ float w_s[kStage];
    __shared__ int cp_s[BWD ? kMaxKK + 1 : 1];
    // slices of the outputs: (channel, slice) by the grid, or a grid of one dimension
    // and all channels of a slice on one XCD (blocks are dealt to them round-robin)
    int ch = blockIdx.x, slice = blockIdx.y;
    if constexpr (MAPPED) {
        const int channels = gridDim.x / slices, whole = slices / 8 * 8;
        const bool tail = (int)blockIdx.x >= whole * channels;
        const int r = tail ? blockIdx.x - whole * channels : blockIdx.x / 8;
        ch = r % channels;
        slice = tail ? whole + r / channels : r / channels * 8 + blockIdx.x % 8;
    }
    const int kk = g.KH * g.KW;
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    int s, e;
    if constexpr (BWD) {  // the column pointers of this channel's KH*KW filter columns (kk <= kMaxKK)
        for (int c = threadIdx.x; c <= kk; c += kThreads) cp_s[c] = ptr[ch * kk + c];
        __syncthreads();
        s = uniform(cp_s[0]);
        e = uniform(cp_s[kk]);
    } else {
        s = ptr[ch];
        e = ptr[ch + 1];
    }
    auto stage = [&](int p0, int n) {
        __syncthreads();  // the previous entries are consumed
        for (int i = threadIdx.x; i < n; i += kThreads) {
            const int q = p0 + i;
            int fc;  // filter position kh * KW + kw
            if constexpr (BWD) {
                int lo = 0, hi = kk - 1;  // last c with cp_s[c] <= q
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (cp_s[mid] <= q) lo = mid; else hi = mid - 1;
                }
                fc = lo;
                map_s[i] = idx[q] * g.OH * g.OW;
            } else {
                const int col = idx[q], ci = col / kk;
                fc = col - ci * kk;
                map_s[i] = ci * g.H * g.W;
            }
            const int kh = fc / g.KW;
            khw_s[i] = (kh << 16) | (fc - kh * g.KW);
            w_s[i] = vals[q];
        }
        __syncthreads();
    };
    const bool one_pass = e - s <= kStage;
    if (one_pass) stage(s, e - s);
    const int ow_ = BWD ? g.W : g.OW, npos = ow_ * (BWD ? g.H : g.OH);
    // (a uniform trip count: every wave of the workgroup stages)
    for (int t0 = slice * (kThreads / kWave); t0 < tasks; t0 += (MAPPED ? slices : gridDim.y) * (kThreads / kWave)) {
        const int t = t0 + wave;
        const bool live = t < tasks;
        const int pg = t / chunks, b = (t - pg * chunks) * (kWave * VEC) + lane * VEC;
        const bool active = live && b < B;
        const int bl = active ? b : 0;
        int oh[kPB], ow[kPB];
        typename V::T acc[kPB];
#pragma unroll
        for (int j = 0; j < kPB; ++j) {
            const int pos = pg * kPB + j;
            oh[j] = pos / ow_;
            ow[j] = pos - oh[j] * ow_;
            acc[j] = V::zero();
        }
        for (int p0 = s; p0 < e; p0 += kStage) {
            const int n = min(kStage, e - p0);
            if (!one_pass) stage(p0, n);
            if (!live) continue;
            for (int e0 = 0; e0 < n; e0 += kWave) {
                const int i = e0 + lane < n ? e0 + lane : n - 1;
                const int kh = khw_s[i] >> 16, kw = khw_s[i] & 0xffff, map = map_s[i];
                const float w = w_s[i];
                int row[kPB];  // this lane's entry: its input row for position j, -1 outside the map
                uint64_t todo = 0;
#pragma unroll
                for (int j = 0; j < kPB; ++j) {
                    bool ok = e0 + lane < n && pg * kPB + j < npos;
                    int r, c;
                    if constexpr (BWD) {
                        const int th = oh[j] + g.PH - kh, tw = ow[j] + g.PW - kw;  // oh*SH, ow*SW
                        r = th;
                        c = tw;
                        if (g.SH > 1 || g.SW > 1) {
                            r = th / g.SH;
                            c = tw / g.SW;
                            ok = ok && r * g.SH == th && c * g.SW == tw;
                        }
                        ok = ok && th >= 0 && tw >= 0 && r < g.OH && c < g.OW;
                        row[j] = ok ? map + r * g.OW + c : -1;
                    } else {
                        r = oh[j] * g.SH - g.PH + kh;
                        c = ow[j] * g.SW - g.PW + kw;
                        ok = ok && r >= 0 && r < g.H && c >= 0 && c < g.W;
                        row[j] = ok ? map + r * g.W + c : -1;
                    }
                    todo |= wave_ballot(ok);
                }
                while (todo) {
                    typename V::T x[kNB][kPB];
                    int rr[kNB][kPB];
                    float ww[kNB];
#pragma unroll
                    for (int u = 0; u < kNB; ++u) {
                        const int src = todo ? __builtin_ctzll(todo) : 0;
                        const bool have = todo != 0;
                        todo &= todo - 1;
                        ww[u] = lane_bcast(w, src);
#pragma unroll
                        for (int j = 0; j < kPB; ++j) {
                            rr[u][j] = have ? lane_bcast(row[j], src) : -1;
                            x[u][j] = V::load(in + (rr[u][j] >= 0 ? rr[u][j] : 0) * ldi + bl);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < kNB; ++u)
#pragma unroll
                        for (int j = 0; j < kPB; ++j)
                            if (rr[u][j] >= 0) V::fma(acc[j], ww[u], x[u][j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kPB; ++j)
            if (active && pg * kPB + j < npos)
                V::store(out + ((int64_t)ch * npos + pg * kPB + j) * ldo + b, acc[j]);
    }
}

// im2col: row r = (ci, kh, kw) of the lowered operand, flattened columns
// f = pos*B + b; VEC consecutive f per thread (one position).
template <int VEC>
__global__ __launch_bounds__(kThreads) void im2col_kernel(geom_t g, int B, const float *__restrict__ X,
                                                          int64_t ldx, float *__restrict__ Xc, int64_t ldc,
                                                          int slices) {
    typedef vec_t<VEC> V;
    const int r = blockIdx.x / slices;
    const int slice = blockIdx.x - r * slices;
    const int64_t F = (int64_t)g.OH * g.OW * B;
    const int64_t f = ((int64_t)slice * kThreads + threadIdx.x) * VEC;
    if (f >= F) return;
    const int pos = (int)(f / B);
    const int b = (int)(f - (int64_t)pos * B);
    const int oh = pos / g.OW, ow = pos - oh * g.OW;
    const int ci = r / (g.KH * g.KW);
    const int kh = (r / g.KW) % g.KH, kw = r % g.KW;
    const int ih = oh * g.SH - g.PH + kh, iw = ow * g.SW - g.PW + kw;
    typename V::T v = V::zero();
    if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W) v = V::load(X + ((int64_t)(ci * g.H + ih) * g.W + iw) * ldx + b);
    V::store(Xc + (int64_t)r * ldc + f, v);
}

template <int VEC>
__global__ __launch_bounds__(kThreads) void maxpool_kernel(geom_t g, int B, const float *__restrict__ X,
                                                           int64_t ldx, float *__restrict__ Y, int64_t ldy,
                                                           int slices) {
    typedef vec_t<VEC> V;
    const int c = blockIdx.x / slices;
    const int slice = blockIdx.x - c * slices;
    const int64_t F = (int64_t)g.OH * g.OW * B;
    const int64_t f = ((int64_t)slice * kThreads + threadIdx.x) * VEC;
    if (f >= F) return;
    const int pos = (int)(f / B);
    const int b = (int)(f - (int64_t)pos * B);
    const int oh = pos / g.OW, ow = pos - oh * g.OW;
    const float *x0 = X + ((int64_t)(c * g.H + oh * g.SH) * g.W + ow * g.SW) * ldx + b;
    typename V::T m = V::load(x0);
    for (int i = 0; i < g.KH; ++i)
        for (int j = 0; j < g.KW; ++j) V::vmax(m, V::load(x0 + ((int64_t)i * g.W + j) * ldx));
    V::store(Y + ((int64_t)(c * g.OH + oh) * g.OW + ow) * ldy + b, m);
}

bool vec4_ok(int B, int64_t lda, const void *a, int64_t ldb, const void *b) {
    return B % 4 == 0 && lda % 4 == 0 && ldb % 4 == 0 && aligned16(a) && aligned16(b);
}

int64_t slices_of(int64_t F, int vec) { return ceil_div(F, (int64_t)kThreads * vec); }

constexpr int64_t kMaxGridX = 0x7fffffff;
// blocks per channel: one per slice (many short blocks keep the most gathers in
// flight; fewer blocks walking several slices each measured slower), at most
// 65535, the rest walked by the blocks' slice loop
int64_t slice_blocks(int64_t slices, int64_t channels) {
    (void)channels;
    return slices < 65535 ? (slices < 1 ? 1 : slices) : 65535;
}

// Floats per lane of the wave kernel, 0 for the thread-per-output kernels: the
// widest vector the alignment allows that keeps three quarters of the lanes
// busy, else single floats where that keeps more than half of them busy.
// Forward, vectors of four against four a thread in the other kernel, or single
// floats against single floats: with narrower vectors than the other kernel's
// it was slower (128 -> 40 channels 20 x 20, batch 128: 212 -> 263 us).  Backward
// the other kernel's index arithmetic costs more than that (527 -> 301), up to a
// batch of 40 in 64 lanes (158 -> 198).
int wave_vec(bool bwd, int B, int64_t lda, const void *a, int64_t ldb, const void *b) {
    const bool v4 = vec4_ok(B, lda, a, ldb, b);
    for (int v = 4; v >= 1; v /= 2) {
        if (v > 1 && (B % v || lda % v || ldb % v || (uintptr_t)a % (4 * v) || (uintptr_t)b % (4 * v))) continue;
        const double used = (double)B / (double)(ceil_div(B, kWave * v) * kWave * v);
        if (used >= 0.75 || (v == 1 && used >= 0.55 && B > kWave)) return bwd || v == 4 || !v4 ? v : 0;
    }
    return 0;
}

// Backward, fewer floats a lane than the other kernel's four.  Single floats: a
// wave per position is four times the waves of the other kernel, which pays
// where a channel's entries are many (its index arithmetic) or the positions few
// (its waves).  Thread per output, wave, us: 256 -> 64 channels, 14 x 14, 1 x 1
// filters at 10 %, batch 48 19.0, 33.2, batch 64 22.9, 33.4; 20 -> 16, 28 x 28, 1 x 1 at
// 5 %, batch 64 6.9, 10.6; 16 -> 32, 28 x 28, 2 x 2 at 10 %, batch 48 12.7, 15.2; 64 ->
// 256, 14 x 14, 1 x 1 at 10 %, batch 64 22.8, 20.2; 20 -> 512, 7 x 7, 1 x 1 at 10 %,
// batch 48 22.5, 7.5.  Strides are divisions in the other kernel.  And a small grid is
// latency, of which the other kernel has more: 64 -> 128, 8 x 8, 1 x 1, stride 2, padding 2
// at 3 %, batch 48 6.7, 4.4; 40 -> 16, 14 x 14, 1 x 1 at 5 %, batch 64 5.5, 6.2.
//
// Pairs: twice the waves, so only where a twelfth of the lanes is idle, the grid
// is full, the entries are fewer still and no stride divides (128 -> 64, 28 x 28, 1 x 1,
// stride 2, batch 320 166, 145).  256 -> 64, 14 x 14, 1 x 1 at 5 %, batch 96 22.9,
// 29.6, batch 300 60.5, 82.4; 20 -> 16, 28 x 28, 1 x 1 at 5 %, batch 112 10.1, 11.1, batch 300
// 20.9, 27.8; 20 -> 6, 14 x 14, 1 x 1 at 10 %, batch 300 7.9, 8.9, batch 96 5.2, 4.4; 64 -> 256,
// 14 x 14, 1 x 1 at 5 %, batch 100 17.6, 15.2; 64 -> 64 at 5 %, batch 128 10.4, 9.5.
bool short_rows(const geom_t &g, int vec, int B, int64_t nnz) {
    const double entries = (double)nnz / (g.C > 0 ? g.C : 1), positions = (double)g.C * g.H * g.W;
    const bool strided = g.SH > 1 || g.SW > 1;
    if (positions * B < (vec == 1 ? 350e3 : 500e3)) return false;
    if (vec == 1) return entries * (B >= kWave || strided ? 1000 : 300) < positions;
    const bool idle = 12 * (int64_t)B <= 11 * ceil_div(B, kWave * vec) * kWave * vec;
    return idle && !strided && entries * 3000 < positions;
}

template <bool BWD>
hipError_t launch_wave(int vec, const geom_t &g, int channels, int B, const int *ptr, const int *idx, const float *vals,
                       const float *in, int64_t ldi, float *out, int64_t ldo, hipStream_t s) {
    const int64_t npos = BWD ? (int64_t)g.H * g.W : (int64_t)g.OH * g.OW;
    const int chunks = (int)ceil_div(B, kWave * vec);
    const int64_t tasks = ceil_div(npos, wave_positions(BWD)) * chunks;
    if (tasks > INT32_MAX - 65535 * 4 || channels > kMaxGridX) return hipErrorInvalidConfiguration;
    // The channels of a slice read the same input rows.  Where the input is more
    // than a few L2s they have to do so on one XCD at a time, or each fetches all of
    // it: forward 256 -> 64 channels, 14 x 14, 1 x 1 filters at 40 %, batch 1024: 515 us by
    // (channel, slice), 185 mapped, 357 with a thread per output; 64 -> 128, 3 x 3 at 5 %, batch 1024: 224,
    // 111, 174.  Smaller inputs gain nothing (12.8 MB: 46.4 -> 48.9; 16 MB: 7.0 -> 7.4) and strided
    // backward products leave whole slices without work (46 -> 67).
    const int64_t all = ceil_div(tasks, kThreads / kWave);
    const bool map = !BWD && (double)g.C * g.H * g.W * B * sizeof(float) > 24e6 && all * channels < (int64_t)1 << 24;
    const int64_t slices = map ? all : slice_blocks(all, channels);
    const dim3 grid = map ? dim3((unsigned)(slices * channels)) : dim3((unsigned)channels, (unsigned)slices);
    auto launch = [&](auto v) {
        constexpr int VEC = decltype(v)::value;
        const auto kernel = map ? conv_wave_kernel<VEC, BWD, !BWD> : conv_wave_kernel<VEC, BWD, false>;
        kernel<<<grid, kThreads, 0, s>>>(g, B, chunks, ptr, idx, vals, in, ldi, out, ldo, (int)tasks, (int)slices);
    };
    if (vec == 4)
        launch(std::integral_constant<int, 4>{});
    else if (vec == 2)
        launch(std::integral_constant<int, 2>{});
    else
        launch(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

}  // namespace

bool conv_out_dims(const conv_geom &g, int *OH, int *OW) {
    if (g.C < 1 || g.H < 1 || g.W < 1 || g.KH < 1 || g.KW < 1 || g.SH < 1 || g.SW < 1 || g.PH < 0 || g.PW < 0)
        return false;
    if (g.KH > 0xffff || g.KW > 0xffff) return false;
    if ((int64_t)g.KH * g.KW > kMaxKK) return false;
    if (g.H + 2 * g.PH < g.KH || g.W + 2 * g.PW < g.KW) return false;
    const geom_t t = to_geom(g);
    *OH = t.OH;
    *OW = t.OW;
    return true;
}

hipError_t launch_conv_fwd(const conv_geom &cg, int N, int B, const int *ptr, const int *idx,
                           const float *vals, const float *X, int64_t ldx, float *Y, int64_t ldy,
                           hipStream_t s) {
    const geom_t g = to_geom(cg);
    const int64_t F = (int64_t)g.OH * g.OW * B;
    if (N == 0 || F == 0) return hipSuccess;
    if (const int vec = wave_vec(false, B, ldx, X, ldy, Y))
        return launch_wave<false>(vec, g, N, B, ptr, idx, vals, X, ldx, Y, ldy, s);
    const bool v4 = vec4_ok(B, ldx, X, ldy, Y);
    const int64_t sl = slices_of(F, v4 ? 4 : 1);
    if (sl > INT32_MAX || N > kMaxGridX) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)N, (unsigned)slice_blocks(sl, N));
    if (v4)
        conv_fwd_kernel<4><<<grid, kThreads, 0, s>>>(g, B, ptr, idx, vals, X, ldx, Y, ldy, (int)sl);
    else
        conv_fwd_kernel<1><<<grid, kThreads, 0, s>>>(g, B, ptr, idx, vals, X, ldx, Y, ldy, (int)sl);
    return hipGetLastError();
}

hipError_t launch_conv_bwd_data(const conv_geom &cg, int N, int B, int64_t nnz, const int *col_ptr,
                                const int *row_idx, const float *vals_t, const float *dY, int64_t ldy, float *dX, int64_t ldx,
                                hipStream_t s) {
    const geom_t g = to_geom(cg);
    const int64_t F = (int64_t)g.H * g.W * B;
    if (F == 0) return hipSuccess;
    (void)N;
    const bool v4 = vec4_ok(B, ldy, dY, ldx, dX);
    const int vec = wave_vec(true, B, ldy, dY, ldx, dX);
    if (vec > 0 && !(vec <= 2 && v4 && short_rows(g, vec, B, nnz)))
        return launch_wave<true>(vec, g, g.C, B, col_ptr, row_idx, vals_t, dY, ldy, dX, ldx, s);
    const int64_t sl = slices_of(F, v4 ? 4 : 1);
    if (sl > INT32_MAX || g.C > kMaxGridX) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)g.C, (unsigned)slice_blocks(sl, g.C));
    if (v4)
        conv_bwd_kernel<4><<<grid, kThreads, 0, s>>>(g, B, col_ptr, row_idx, vals_t, dY, ldy, dX, ldx, (int)sl);
    else
        conv_bwd_kernel<1><<<grid, kThreads, 0, s>>>(g, B, col_ptr, row_idx, vals_t, dY, ldy, dX, ldx, (int)sl);
    return hipGetLastError();
}

hipError_t launch_im2col(const conv_geom &cg, int B, const float *X, int64_t ldx, float *Xc, int64_t ldc,
                         hipStream_t s) {
    const geom_t g = to_geom(cg);
    const int64_t F = (int64_t)g.OH * g.OW * B;
    const int64_t R = (int64_t)g.C * g.KH * g.KW;
    if (F == 0 || R == 0) return hipSuccess;
    const bool v4 = vec4_ok(B, ldx, X, ldc, Xc);
    const int64_t sl = slices_of(F, v4 ? 4 : 1);
    if (sl * R > INT32_MAX) return hipErrorInvalidConfiguration;
    const unsigned grid = (unsigned)(sl * R);
    if (v4)
        im2col_kernel<4><<<grid, kThreads, 0, s>>>(g, B, X, ldx, Xc, ldc, (int)sl);
    else
        im2col_kernel<1><<<grid, kThreads, 0, s>>>(g, B, X, ldx, Xc, ldc, (int)sl);
    return hipGetLastError();
}

hipError_t launch_maxpool_fwd(const conv_geom &cg, int B, const float *X, int64_t ldx, float *Y, int64_t ldy,
                              hipStream_t s) {
    const geom_t g = to_geom(cg);
    const int64_t F = (int64_t)g.OH * g.OW * B;
    if (F == 0) return hipSuccess;
    const bool v4 = vec4_ok(B, ldx, X, ldy, Y);
    const int64_t sl = slices_of(F, v4 ? 4 : 1);
    if (sl * g.C > INT32_MAX) return hipErrorInvalidConfiguration;
    const unsigned grid = (unsigned)(sl * g.C);
    if (v4)
        maxpool_kernel<4><<<grid, kThreads, 0, s>>>(g, B, X, ldx, Y, ldy, (int)sl);
    else
        maxpool_kernel<1><<<grid, kThreads, 0, s>>>(g, B, X, ldx, Y, ldy, (int)sl);
    return hipGetLastError();
}

}  // namespace l1csr
