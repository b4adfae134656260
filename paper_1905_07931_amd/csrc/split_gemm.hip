// C[M][Nn] = A[M][Kr] . B[Nn][Kr]^T in fp32 accuracy on the bf16 matrix cores
// (v_mfma_f32_32x32x16_bf16): every fp32 operand is split into bf16 parts,
// packed once per call in the order the matrix cores read them.
//
// Parts.  Three (hi, mid, lo): hi = bf16(x), mid = bf16(x - hi), lo = bf16(x -
// hi - mid), each to nearest even; 3 x 8 significand bits hold the 24 of x, so
// hi + mid + lo = x.  A product takes the six terms down to 2^-16 of it (hi hi,
// mid hi, hi mid, mid mid, lo hi, hi lo); each is exact in fp32 and summed in
// fp32.  What is left out (mid lo, lo mid, lo lo) is at most 2^-23 of |a b|, of
// random sign.  16 products are summed per instruction instead of 2, so there
// are fewer roundings than in the fp32 instruction's sum: at 4096 x 9216 x
// 1024 the result is 1.8e-7 off the 64-bit one (2-norm), 5.7e-7 with
// v_mfma_f32_32x32x2_f32.  The bf16 pipe is 16x the fp32 one, so six products
// have 2.7x its peak.  Two parts (hi, lo) with three terms are the BF16X3
// arithmetic (2^-16 left out).
//
// The parts are those of 2^24 x, and a sum is scaled back by 2^-48 (both exact,
// but for a result that is itself subnormal): the last bit of the smallest fp32
// number, 2^-149, then lies at 2^-125, so no part underflows, whatever stands
// beside it.  The parts hold every |x| up to 2^28, with which no sum of 2^22
// products overflows (2^126).  The pack kernel flags every (32-row group,
// 256-index block) that holds a NaN, an infinity or an |x| above 2^28 and leaves
// its parts zero; a tile adds the products of its flagged blocks (both operands'
// groups over those 256 indices) from the operands themselves, by the fp32
// matrix-core instruction, or over a CSR operand entry by entry.  What that
// costs, us per call for ordinary operands, one infinity in X, and 2 % of X
// infinite (a flag on every block): forward product 4096 x 4096 x 512 at 20 %
// 128, 197, 1450 (7000 and 8200 with whole tiles left to a thread per column),
// masked gradient there 102, 115, 215; gradient 4096 x 9216 x 1024 399, 410, 821.
//
// What bounds it: the matrix pipe, and through it the power limit.  With every
// CU's matrix pipe 71 % busy the shader clock falls to 1.64 GHz (2.38 GHz under
// the fp32 instruction), 1.2-1.27 PFLOP/s of bf16 at 4096 x 9216 x 1024, where
// a large bf16 library product reaches 1.12.
#include <cmath>

#include "common.hpp"
#include "launch.hpp"
#include "prox_epilogue.hpp"

namespace l1csr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void sg_lds_void;

constexpr int kGroup = 32;         // rows of a packed group
constexpr int kStep = 16;          // reduction indices of a packed block
constexpr int kBlockBytes = 1024;  // one part of a (group, step): 64 lanes x 16 bytes
constexpr int kPackK = 256;        // reduction indices of a pack workgroup (one flag)
constexpr float kPartMax = 0x1p28f, kPartScale = 0x1p24f;
constexpr float kSumScale = 1.f / (kPartScale * kPartScale);

// A packed operand: [group][step][part][lane][8] bf16.  Lane l of a block holds
// row l % 32 of the group and reduction indices 8 (l / 32) .. + 7 of the step,
// the operand fragment of one MFMA: the copy into LDS and the fragment reads
// are both linear in the lane (whole cache lines, no bank conflicts, no
// swizzle).  Rows and indices past the matrix are zeros.
struct packed {
    char *data;
    int *flags;  // [group][kPackK block]: not exact in parts
    int groups, steps, kblocks;
};

int64_t packed_bytes(int rows, int kr, int np) {
    return ceil_div(rows, kGroup) * ceil_div(kr, kStep) * (int64_t)(np * kBlockBytes);
}
int64_t flag_bytes(int rows, int kr) {
    return ceil_div(ceil_div(rows, kGroup) * ceil_div(kr, kPackK) * (int64_t)sizeof(int), 256) * 256;
}
// carves rows x kr out of p (advanced past it)
packed carve_packed(char *&p, int rows, int kr, int np) {
    packed o;
    o.groups = (int)ceil_div(rows, kGroup);
    o.steps = (int)ceil_div(kr, kStep);
    o.kblocks = (int)ceil_div(kr, kPackK);
    o.data = p;
    p += packed_bytes(rows, kr, np);
    o.flags = reinterpret_cast<int *>(p);
    p += flag_bytes(rows, kr);
    return o;
}

template <int NP>
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&p)[NP]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float r = x[e] * kPartScale;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const __bf16 h = (__bf16)r;
            p[q][e] = h;
            r -= (float)h;
        }
    }
}

// What the packing of 8 values shares: their parts stored, magnitudes tracked
template <int NP>
__device__ __forceinline__ void pack8(const float (&x)[8], unsigned &mx, char *d) {
#pragma unroll
    for (int e = 0; e < 8; ++e) mx = max(mx, __float_as_uint(x[e]) & 0x7fffffffu);
    bf16x8 p[NP];
    split8<NP>(x, p);
#pragma unroll
    for (int q = 0; q < NP; ++q) *reinterpret_cast<bf16x8 *>(d + q * kBlockBytes) = p[q];
}

// Ends the workgroup's pack of block kb of group g: stores its flag and zeroes the
// parts of a flagged block.  rowmax: the 32 rows' magnitudes in LDS (zeroed, a
// barrier behind it).
template <int NP>
__device__ __forceinline__ void store_flag(unsigned *rowmax, unsigned mx, const packed &o, int g, int kb) {
    const int lane = threadIdx.x & 63;
    atomicMax(&rowmax[lane & 31], mx);
    __syncthreads();  // (the waves' parts are stored)
    if (threadIdx.x >= kWave) return;
    const bool odd = __ballot(rowmax[lane & 31] > __float_as_uint(kPartMax)) != 0ull;
    if (lane == 0) o.flags[g * o.kblocks + kb] = odd;
    if (!odd) return;
    const int s0 = kb * (kPackK / kStep), n = min(kPackK / kStep, o.steps - s0) * NP;
    char *d = o.data + ((int64_t)g * o.steps + s0) * (NP * kBlockBytes) + lane * 16;
    for (int q = 0; q < n; ++q) *reinterpret_cast<bf16x8 *>(d + q * kBlockBytes) = bf16x8{};
}

// one operand of a pack launch: rows of a row-major fp32 matrix, the reduction
// index contiguous (v4: 16-byte aligned rows)
struct pack_src {
    const float *p;
    int64_t ld;
    int rows, v4;
    packed out;
};

// Both operands of a product in one launch.  A workgroup takes one 32-row group
// and 256 reduction indices; a wave a step of 16 at a time: lane l reads the 8
// floats of its row and half and writes its 16 bytes of each part, 1 KB a store.
// Memory-bound: 4 bytes read and 2 NP written per element, 22.5 us for 54.5 MB
// in and 82 MB out (6.0 TB/s) with three parts at 4096 + 9216 rows of 1024.
template <int NP>
__global__ __launch_bounds__(256) void pack_rows_kernel(pack_src s0, pack_src s1, int kr) {
    __shared__ unsigned rowmax[kGroup];
    const bool first = (int)blockIdx.x < s0.out.groups;
    const pack_src s = first ? s0 : s1;
    const int g = first ? blockIdx.x : blockIdx.x - s0.out.groups;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < kGroup) rowmax[threadIdx.x] = 0u;
    __syncthreads();
    const int row = g * kGroup + (lane & 31);
    const float *src = s.p + (int64_t)row * s.ld;
    unsigned mx = 0u;  // magnitudes as ordered integers; NaN above infinity
#pragma unroll
    for (int i = 0; i < kPackK / kStep / 4; ++i) {
        const int st = blockIdx.y * (kPackK / kStep) + i * 4 + wave;
        if (st >= s.out.steps) break;
        const int k = st * kStep + (lane >> 5) * 8;
        float x[8];
        if (s.v4 && row < s.rows && k + 7 < kr) {
            const float4 a = *reinterpret_cast<const float4 *>(src + k);
            const float4 b = *reinterpret_cast<const float4 *>(src + k + 4);
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
            x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = row < s.rows && k + e < kr ? src[k + e] : 0.f;
        }
        pack8<NP>(x, mx, s.out.data + ((int64_t)g * s.out.steps + st) * (NP * kBlockBytes) + lane * 16);
    }
    store_flag<NP>(rowmax, mx, s.out, g, blockIdx.y);
}

// Both operands of a sparse product in one launch: a CSR matrix (the first
// groups) and the transpose of the dense operand X [Kr][ldx], whose packed rows
// are its columns.  A workgroup takes a 32-row group and 256 reduction indices
// of either.  The CSR part: the rows' first entries at both ends of the index
// range are searched for, the entries between them scattered into a zeroed LDS
// tile, which is packed.  The X part: a lane's 8 values are 8 rows apart, 32 lanes
// read 128 consecutive bytes of each.  Memory-bound on the parts written (6
// bytes per weight, zeros included): 25 us at 4096 x 4096 x 512 and 5 % stored
// (108 MB, 4.4 TB/s), 42 us at 50 % (180 MB, 4.3 TB/s).
constexpr int kCsrStride = kPackK + 4;  // floats: 16-byte reads of 32 rows spread over the banks

__global__ __launch_bounds__(256) void pack_spmm_kernel(int n_rows, const int *__restrict__ ptr,
                                                        const int *__restrict__ idx, const float *__restrict__ vals,
                                                        packed A, const float *__restrict__ X, int64_t ldx, int Kr,
                                                        int cols, packed B) {
    __shared__ unsigned rowmax[kGroup];
    __shared__ __attribute__((aligned(16))) float tile[kGroup * kCsrStride];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < kGroup) rowmax[threadIdx.x] = 0u;
    unsigned mx = 0u;
    const int kb = blockIdx.y, k0 = kb * kPackK;
    if ((int)blockIdx.x >= A.groups) {  // X
        const int g = blockIdx.x - A.groups;
        const int col = g * kGroup + (lane & 31);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPackK / kStep / 4; ++i) {
            const int st = kb * (kPackK / kStep) + i * 4 + wave;
            if (st >= B.steps) break;
            const int k = st * kStep + (lane >> 5) * 8;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = col < cols && k + e < Kr ? X[(int64_t)(k + e) * ldx + col] : 0.f;
            pack8<3>(x, mx, B.data + ((int64_t)g * B.steps + st) * (3 * kBlockBytes) + lane * 16);
        }
        store_flag<3>(rowmax, mx, B, g, kb);
        return;
    }
    const int g = blockIdx.x;
    for (int i = threadIdx.x; i < kGroup * kCsrStride / 4; i += 256)
        reinterpret_cast<float4 *>(tile)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    // eight lanes per row: the row's first entries at or past k0 and k0 + 256,
    // eight probes a round (four dependent loads for 4096 entries, not twelve)
    const int r = threadIdx.x >> 3, j = threadIdx.x & 7, row = g * kGroup + r;
    int lo0 = 0, hi0 = 0;
    if (row < n_rows) {
        lo0 = ptr[row];
        hi0 = ptr[row + 1];
    }
    int lo1 = lo0, hi1 = hi0;
    while (__ballot(lo0 < hi0 || lo1 < hi1)) {
        auto probe = [&](int &lo, int &hi, int target) {
            const int n = hi - lo;
            auto at = [&](int q) { return lo + (int)((unsigned)n * (unsigned)(q + 1) / 9u); };  // n < 2^28
            const bool less = n > 0 && idx[at(j)] < target;
            const int c = __popcll((__ballot(less) >> (lane & 56)) & 0xffull);
            if (n > 0) {
                const int nlo = c > 0 ? at(c - 1) + 1 : lo, nhi = c < 8 ? at(c) : hi;
                lo = nlo;
                hi = nhi;
            }
        };
        probe(lo0, hi0, k0);
        probe(lo1, hi1, k0 + kPackK);
    }
    __syncthreads();
    for (int p0 = lo0 + j; p0 < lo1; p0 += 32) {  // four entries a lane in flight
        int c[4];
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int p = p0 + 8 * u;
            c[u] = p < lo1 ? idx[p] - k0 : -1;
            v[u] = p < lo1 ? vals[p] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((unsigned)c[u] < (unsigned)kPackK) tile[r * kCsrStride + c[u]] = v[u];  // (columns ascend in a row)
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPackK / kStep / 4; ++i) {
        const int st = kb * (kPackK / kStep) + i * 4 + wave;
        if (st >= A.steps) break;
        const float4 *t = reinterpret_cast<const float4 *>(tile + (lane & 31) * kCsrStride +
                                                           (i * 4 + wave) * kStep + (lane >> 5) * 8);
        const float4 a = t[0], b = t[1];
        const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        pack8<3>(x, mx, A.data + ((int64_t)g * A.steps + st) * (3 * kBlockBytes) + lane * 16);
    }
    store_flag<3>(rowmax, mx, A, g, kb);
}

__device__ __forceinline__ floatx16 mfma16(bf16x8 a, bf16x8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// One 1 KB block global -> LDS (16 bytes per lane), base and lds wave-uniform.
// As an instruction of its own rather than the builtin: the compiler orders the
// builtin's loads against the reads of the other buffers and waited for the
// loads just issued (vmcnt(0)) in one step of three.  It writes no register;
// wait_vm() below counts it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // m0 is reserved: the clobber orders it, nothing keeps it
__device__ __forceinline__ void dma16(const char *base, unsigned off, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

template <int N>
__device__ __forceinline__ void wait_vm() {  // at most N vector memory operations and no LDS access outstanding
    static_assert(N < 16, "low field only");
    __builtin_amdgcn_s_waitcnt(0x0070 | N);
}

// The tile: 128 x 128, 2 x 2 waves of 64 x 64 (2 x 2 MFMA tiles each), a step of
// 16 reduction indices a time.  A step is 4 + 4 groups of NP blocks (24 KB with
// three parts), three steps in LDS (72 KB): two workgroups share a CU, so one's
// epilogue runs under the other's products.  Per step a wave reads 4 NP
// fragments for 24 (NP = 2: 12) MFMAs.  Larger tiles and waves (256 x 288 with
// 12 waves, 256 x 256 with 8 or 16, 128 x 256, 128 x 128 of two waves) measured
// 400-450 us at 4096 x 9216 x 1024 against 365-377 us: the pipe is held by
// power, not by LDS reads, and the smaller tile wastes least at the edges.
constexpr int TM = 2, TN = 2, WM = 2, WN = 2;
constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN, NT = 64 * WM * WN;
constexpr int RGA = TM * WM, RGB = TN * WN;  // groups of a tile

enum {
    kEpiStore = 0,  // C
    kEpiProx = 1,   // Z = S_t(W - eta C) and its word counts
    kEpiMask = 2,   // C's entries on W's pattern, in CSR order
    kEpiSpmm = 3    // C; A is a packed CSR matrix, B a packed transpose
};

// How a sum is accumulated over the steps (relative error against 64 bits,
// 2-norm, at 1024 / 512 reduction indices; every rounding of the running sum
// costs 2^-25 of it, and the five small terms would each cause one):
//   one set of registers                                     4.9e-7 / 3.5e-7
//   the five small terms in a set of their own               1.8e-7 / 1.2e-7
//   that, and the large terms moved to a third set every six
//   steps (its chain and theirs are then both short)         8.6e-8 / 7.5e-8
// The sums that a kernel replaces set which one it needs: a row of fp32 matrix
// instructions 5.7e-7 / 4.1e-7 (the dense gradient: two sets, since a product
// that the fp32 tiles split into two ranges may be whole here; two parts: one,
// their 2^-16 decides), a sequential fp32 row sum 3-5e-7 (the sparse products: two), a tree over 64 lanes 8.5e-8 (the
// masked gradient: three).  The second set is free (353 and 354 us at 4096 x
// 9216 x 1024), the third costs 3 %.
enum { kAccOne = 1, kAccSmall = 2, kAccTree = 3 };
constexpr int kTreeSteps = 6;  // a multiple of the three steps in LDS

struct gemm_args {
    int M, Nn, Kr;                // sizes (Kr: all reduction indices)
    packed A, B;
    const float *a32, *b32;       // the operands themselves, for flagged blocks
    int64_t lda, ldb;
    int a_v4, b_v4;               // their rows are 16-byte aligned
    int tiles_m, tiles_n;
    int split_steps;              // steps per split (blockIdx.y); the splits' C are M * ldc apart
    float *C;
    int64_t ldc;
    prox_epi P;                   // (kEpiMask: mask, pos and kw; C is the entry array)
    const int *ptr, *idx;         // kEpiSpmm: A as CSR, b32 [Kr][ldb]
    const float *vals;
};

template <int NP, int EPI, int ACC>
__global__ __launch_bounds__(NT, 2) void split_gemm_kernel(gemm_args G) {
    constexpr int PIECES = (RGA + RGB) * NP;     // 1 KB blocks of a step
    constexpr int LPW = PIECES / (NT / kWave);   // loads per wave and step
    static_assert(PIECES % (NT / kWave) == 0, "every wave issues the same number of loads");
    constexpr int SB = PIECES * kBlockBytes;
    __shared__ __attribute__((aligned(16))) char S0[SB];
    __shared__ __attribute__((aligned(16))) char S1[SB];
    __shared__ __attribute__((aligned(16))) char S2[SB];
    // tile order: bands of 8 tile rows walked column by column; each XCD
    // (blocks are dealt round-robin) takes one contiguous range of it, so the
    // tiles it runs at one time share operand rows in its L2
    int tm, tn;
    {
        const int T = G.tiles_m * G.tiles_n, per = (T + 7) / 8;
        const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
        if ((int)(blockIdx.x >> 3) >= per || t >= T) return;
        const int band = t / (8 * G.tiles_n), r = t - band * 8 * G.tiles_n;
        const int h = min(8, G.tiles_m - band * 8);
        tn = r / h;
        tm = band * 8 + (r - tn * h);
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const int wave = uniform(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int wgm = (wave / WN) * TM, wgn = (wave % WN) * TN;  // the wave's first group of A / B in the tile
    const int c0 = blockIdx.y * G.split_steps;
    const int steps = min(G.split_steps, G.A.steps - c0);      // >= 1, or 0 if Kr == 0

    // this wave's blocks of a step: piece p = wave + j * waves
    const char *src[LPW];
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
        const int p = wave + j * (NT / kWave);
        const int g = p / NP, q = p - g * NP;
        const int64_t gs = (int64_t)G.A.steps * (NP * kBlockBytes);
        // groups past the operand: never stored, any data will do
        src[j] = (g < RGA ? G.A.data + min(tm * RGA + g, G.A.groups - 1) * gs
                          : G.B.data + min(tn * RGB + (g - RGA), G.B.groups - 1) * gs) +
                 (int64_t)c0 * (NP * kBlockBytes) + q * kBlockBytes;
    }
    const unsigned l0 = (unsigned)(uintptr_t)(sg_lds_void *)S0 + wave * kBlockBytes;
    const unsigned l1 = (unsigned)(uintptr_t)(sg_lds_void *)S1 + wave * kBlockBytes;
    const unsigned l2 = (unsigned)(uintptr_t)(sg_lds_void *)S2 + wave * kBlockBytes;
    auto load = [&](unsigned dst, int c) {
        const unsigned off = (unsigned)c * (NP * kBlockBytes) + lane * 16;
#pragma unroll
        for (int j = 0; j < LPW; ++j) dma16(src[j], off, dst + j * (NT / kWave) * kBlockBytes);
    };
    // flagged blocks of the tile (the same answer in every wave)
    const int kb0 = c0 / (kPackK / kStep), kb1 = (c0 + steps + kPackK / kStep - 1) / (kPackK / kStep);
    bool odd = false;
    {
        for (int kb = kb0 + (lane >> 3); kb < kb1; kb += 8) {
            const int g = lane & 7;
            const int *f = g < RGA ? G.A.flags + (int64_t)min(tm * RGA + g, G.A.groups - 1) * G.A.kblocks
                                   : G.B.flags + (int64_t)min(tn * RGB + g - RGA, G.B.groups - 1) * G.B.kblocks;
            odd |= f[kb] != 0;
        }
        odd = __ballot(odd) != 0ull;
    }
    static_assert(RGA + RGB == 8, "one lane per group");

    floatx16 acc[TM][TN], small[TM][TN], top[TM][TN];  // (sets that ACC does not use vanish)
    auto each = [&](auto f) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) f(a, b, r);
    };
    each([&](int a, int b, int r) { acc[a][b][r] = small[a][b][r] = top[a][b][r] = 0.f; });

    const int lr = lane & 31, lh = lane >> 5;
    {
        const int oa = wgm * (NP * kBlockBytes) + lane * 16;
        const int ob = (RGA + wgn) * (NP * kBlockBytes) + lane * 16;
        auto compute = [&](const char *cur) {
            bf16x8 af[NP][TM], bf[NP][TN];
#pragma unroll
            for (int q = 0; q < NP; ++q) {
#pragma unroll
                for (int a = 0; a < TM; ++a)
                    af[q][a] = *reinterpret_cast<const bf16x8 *>(cur + oa + (a * NP + q) * kBlockBytes);
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    bf[q][b] = *reinterpret_cast<const bf16x8 *>(cur + ob + (b * NP + q) * kBlockBytes);
            }
            auto term = [&](int qa, int qb) {
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) acc[a][b] = mfma16(af[qa][a], bf[qb][b], acc[a][b]);
            };
            auto small_term = [&](int qa, int qb) {
                if constexpr (ACC == kAccOne) {
                    term(qa, qb);
                } else {
#pragma unroll
                    for (int a = 0; a < TM; ++a)
#pragma unroll
                        for (int b = 0; b < TN; ++b) small[a][b] = mfma16(af[qa][a], bf[qb][b], small[a][b]);
                }
            };
            if constexpr (NP == 2) {
                // the two small terms first, then hi . hi
                small_term(1, 0);
                small_term(0, 1);
                term(0, 0);
            } else {
                // in the order the fragments arrive
                term(0, 0);
                small_term(1, 0);
                small_term(0, 1);
                small_term(1, 1);
                small_term(2, 0);
                small_term(0, 2);
            }
        };
        // step c: its blocks have landed everywhere (the loads of step c + 1 may
        // still be out), and the buffer that the loads of step c + 2 fill was
        // last read in step c - 1, whose reads every wave has finished here
        auto step = [&](int c, const char *cur, unsigned nxt2) {
            if (c + 1 < steps)
                wait_vm<LPW>();
            else
                wait_vm<0>();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (c + 2 < steps) load(nxt2, c + 2);
            compute(cur);
        };
        if (steps > 0) load(l0, 0);
        if (steps > 1) load(l1, 1);
        for (int c = 0; c < steps; c += 3) {
            step(c, S0, l2);
            if (c + 1 < steps) step(c + 1, S1, l0);
            if (c + 2 < steps) step(c + 2, S2, l1);
            if constexpr (ACC == kAccTree)
                if (c % kTreeSteps == kTreeSteps - 3)
                    each([&](int a, int b, int r) {
                        top[a][b][r] += acc[a][b][r];
                        acc[a][b][r] = 0.f;
                    });
        }
        each([&](int a, int b, int r) {
            float sum = acc[a][b][r];
            if constexpr (ACC == kAccTree) sum += top[a][b][r];
            if constexpr (ACC != kAccOne) sum += small[a][b][r];
            acc[a][b][r] = sum * kSumScale;
        });
    }
    if constexpr (EPI != kEpiSpmm) {
        // the flagged blocks: the fp32 instruction, lane half h at indices 4 h .. + 3 of 8
        for (int kb = odd ? kb0 : kb1; kb < kb1; ++kb) {
            int fa[TM], fb[TN], any = 0;
#pragma unroll
            for (int a = 0; a < TM; ++a)
                any |= fa[a] = uniform(G.A.flags[(int64_t)min(tm * RGA + wgm + a, G.A.groups - 1) * G.A.kblocks + kb]);
#pragma unroll
            for (int b = 0; b < TN; ++b)
                any |= fb[b] = uniform(G.B.flags[(int64_t)min(tn * RGB + wgn + b, G.B.groups - 1) * G.B.kblocks + kb]);
            if (!any) continue;
            const int k1 = min(G.Kr, min(c0 + steps, (kb + 1) * (kPackK / kStep)) * kStep);
            auto load4 = [&](const float *p, int64_t ld, int row, int rows, int v4, int k, float (&x)[4]) {
                const float *r = p + row * ld + k;
                if (v4 && row < rows && k + 3 < k1) {
                    const float4 v = *reinterpret_cast<const float4 *>(r);
                    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = row < rows && k + e < k1 ? r[e] : 0.f;
                }
            };
#pragma unroll 2
            for (int k = max(c0, kb * (kPackK / kStep)) * kStep; k < k1; k += 8) {
                float av[TM][4], bv[TN][4];
#pragma unroll
                for (int a = 0; a < TM; ++a)
                    load4(G.a32, G.lda, m0 + (wgm + a) * 32 + lr, G.M, G.a_v4, k + 4 * lh, av[a]);
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    load4(G.b32, G.ldb, n0 + (wgn + b) * 32 + lr, G.Nn, G.b_v4, k + 4 * lh, bv[b]);
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        if (!(fa[a] | fb[b])) continue;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[a][e], bv[b][e], acc[a][b], 0, 0, 0);
                    }
            }
        }
    }
    if constexpr (EPI == kEpiProx) {
        __syncthreads();  // every wave has read its last fragments: the buffers are free
        // the staged index words, then two gather buffers of one MFMA tile (8 KB) per wave
        constexpr int GBF = 2 * 16 * kWave;  // floats per wave
        constexpr int kStageBytes = 8 * BM * (BN / 32);
        constexpr int W0 = (SB - kStageBytes) / (4 * GBF), W1 = SB / (4 * GBF);
        static_assert(W0 >= 1 && W0 + 2 * W1 >= NT / kWave, "gather space");
        int2 *stage = reinterpret_cast<int2 *>(S0);
        prox_stage<BM, BN, NT>(G.P, G.M, m0, n0, stage);
        float *gbuf = wave < W0 ? reinterpret_cast<float *>(S0 + kStageBytes) + wave * GBF
                                : (wave < W0 + W1 ? reinterpret_cast<float *>(S1) + (wave - W0) * GBF
                                                  : reinterpret_cast<float *>(S2) + (wave - W0 - W1) * GBF);
        prox_store<TN, BN, 1, 2>(acc, G.M, G.Nn, m0, n0, wgm * 32, wgn * 32, stage, gbuf, G.C, G.ldc, G.P);
        return;
    }
    // D layout of the 32x32 MFMA: lane l, register r holds
    // row 8*(r/4) + 4*(l/32) + r%4, column l%32 of the 32x32 tile.
    if constexpr (EPI == kEpiMask) {
        // the entries of a row's 32-column word are consecutive in the CSR
        __syncthreads();
        int2 *stage = reinterpret_cast<int2 *>(S0);
        prox_stage<BM, BN, NT>(G.P, G.M, m0, n0, stage);
        const unsigned below = (1u << lr) - 1u;
        each([&](int a, int b, int r) {
            const int2 mp = stage[((wgm + a) * 32 + 8 * (r >> 2) + 4 * lh + (r & 3)) * (BN / 32) + wgn + b];
            const unsigned m = (unsigned)mp.x;
            if ((m >> lr) & 1u) G.C[mp.y + __popc(m & below)] = acc[a][b][r];
        });
        return;
    }
    float *C = G.C + (int64_t)blockIdx.y * G.M * G.ldc;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int col = n0 + (wgn + b) * 32 + lr;
            if (col >= G.Nn) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + (wgm + a) * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                if (row < G.M) C[(int64_t)row * G.ldc + col] = acc[a][b][r];
            }
        }
    if constexpr (EPI == kEpiSpmm) {
        // the flagged blocks: the stored entries of A alone (a zero of the packed
        // copy would turn an infinity of B into NaN), half a wave per row and 32 columns
        if (!odd) return;
        __syncthreads();  // the tile is stored, the LDS buffers are free
        int2 *ends = reinterpret_cast<int2 *>(S0);  // each row's entries in the block
        for (int kb = kb0; kb < kb1; ++kb) {
            const int g = lane & 7;
            const int *f = g < RGA ? G.A.flags + (int64_t)min(tm * RGA + g, G.A.groups - 1) * G.A.kblocks
                                   : G.B.flags + (int64_t)min(tn * RGB + g - RGA, G.B.groups - 1) * G.B.kblocks;
            const unsigned flagged = (unsigned)__ballot(f[kb] != 0) & 0xffu;  // A's groups, then B's
            if (flagged == 0u) continue;  // (the same in every wave)
            const int k0 = max(c0, kb * (kPackK / kStep)) * kStep;
            const int k1 = min(G.Kr, min(c0 + steps, (kb + 1) * (kPackK / kStep)) * kStep);
            __syncthreads();  // the previous block's bounds are consumed
            for (int r = threadIdx.x; r < BM; r += NT) {
                int2 e = make_int2(0, 0);
                if (m0 + r < G.M) {
                    const int end = G.ptr[m0 + r + 1];
                    auto first_at = [&](int lo, int k) {
                        int hi = end;
                        while (lo < hi) {
                            const int mid = lo + (hi - lo) / 2;
                            if (G.idx[mid] < k) lo = mid + 1; else hi = mid;
                        }
                        return lo;
                    };
                    e.x = first_at(G.ptr[m0 + r], k0);
                    e.y = first_at(e.x, k1);
                }
                ends[r] = e;
            }
            __syncthreads();
            for (int it = wave * 2 + lh; it < BM * RGB; it += 2 * (NT / kWave)) {
                const int r = it % BM, cg = it / BM, col = n0 + cg * 32 + lr;
                if (!(((flagged >> (r >> 5)) | (flagged >> (RGA + cg))) & 1u) || col >= G.Nn) continue;
                const int2 e = ends[r];
                if (e.x == e.y) continue;
                float sum = 0.f;
                for (int p0 = e.x; p0 < e.y; p0 += 16) {
                    float v[16], x[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        const int p = min(p0 + u, e.y - 1);
                        v[u] = G.vals[p];
                        x[u] = G.b32[(int64_t)G.idx[p] * G.ldb + col];
                    }
#pragma unroll
                    for (int u = 0; u < 16; ++u)
                        if (p0 + u < e.y) sum = fmaf(v[u], x[u], sum);
                }
                C[(int64_t)(m0 + r) * G.ldc + col] += sum;
            }
        }
    }
}

template <int NP>
hipError_t launch_pack(const pack_src &a, const pack_src &b, int kr, hipStream_t s) {
    dim3 grid((unsigned)(a.out.groups + b.out.groups), (unsigned)a.out.kblocks);
    pack_rows_kernel<NP><<<grid, 256, 0, s>>>(a, b, kr);
    return hipGetLastError();
}

template <int NP, int EPI, int ACC>
hipError_t launch_tiles(gemm_args G, int splits, hipStream_t s) {
    G.tiles_m = (int)ceil_div(G.M, BM);
    G.tiles_n = (int)ceil_div(G.Nn, BN);
    dim3 grid((unsigned)(ceil_div((int64_t)G.tiles_m * G.tiles_n, 8) * 8), (unsigned)splits);
    split_gemm_kernel<NP, EPI, ACC><<<grid, NT, 0, s>>>(G);
    return hipGetLastError();
}

// Ranges of the reduction: as many as give every CU one workgroup (of >= 256
// indices each).  From 129 tiles on a product is whole: partial results that are
// written, added and, without the fused epilogue, read again by the prox cost
// more than the second workgroup on a CU gives.  us for dense_wgrad, prox,
// with the 512 workgroups that the fp32 tiles want -> 256: 503 x 7856 x 736 58.9
// -> 50.6, 73.0 -> 58.6; 1200 x 3000 x 1000 64.8 -> 54.2, 79.8 -> 62.7; BF16X3 1500 x
// 2000 x 600 31.7 -> 28.0, 45.3 -> 37.1; 1024 x 1024 x 1024 29.4 -> 30.4, 34.8 -> 35.1.
wgrad_split split_plan(int N, int K, int B) {
    wgrad_split p{1, B};
    const int64_t tiles = ceil_div(N, BM) * ceil_div(K, BN);
    int64_t s = tiles > 0 ? 256 / tiles : 1;
    s = s < B / 256 ? s : B / 256;
    s = s < 64 ? s : 64;
    if (s < 2) return p;
    const int64_t chunk = ceil_div(ceil_div(B, s), 2 * kStep) * 2 * kStep;
    p.splits = (int)ceil_div(B, chunk);
    p.chunk = (int)chunk;
    return p;
}

// dY . X^T with the operands packed into ws; a product of few tiles splits its
// reduction by split_plan() into partial results behind the packed operands,
// which wgrad_reduce_kernel adds in order
template <int NP, int EPI>
hipError_t wgrad(int N, int K, int B, const float *dY, int64_t ldy, const float *X, int64_t ldx, float *C,
                 int64_t ldc, const prox_epi &P, void *ws, hipStream_t s) {
    char *p = static_cast<char *>(ws);
    gemm_args G{};
    G.A = carve_packed(p, N, B, NP);
    G.B = carve_packed(p, K, B, NP);
    G.a_v4 = ldy % 4 == 0 && aligned16(dY); G.b_v4 = ldx % 4 == 0 && aligned16(X);
    hipError_t e = launch_pack<NP>(pack_src{dY, ldy, N, G.a_v4, G.A},
                                   pack_src{X, ldx, K, G.b_v4, G.B}, B, s);
    if (e != hipSuccess) return e;
    G.M = N; G.Nn = K; G.Kr = B;
    G.a32 = dY; G.lda = ldy; G.b32 = X; G.ldb = ldx;
    G.split_steps = G.A.steps;
    G.C = C; G.ldc = ldc; G.P = P;
    // three parts: the small terms apart, which makes a whole sum at least as
    // exact as the fp32 instruction's over half as many indices
    constexpr int ACC = NP == 3 ? kAccSmall : kAccOne;
    const wgrad_split w = split_plan(N, K, B);
    if (w.splits == 1) return launch_tiles<NP, EPI, ACC>(G, 1, s);
    float *parts = reinterpret_cast<float *>(p);
    G.split_steps = w.chunk / kStep;
    G.C = parts; G.ldc = K;
    e = launch_tiles<NP, kEpiStore, ACC>(G, w.splits, s);
    if (e != hipSuccess) return e;
    return launch_wgrad_reduce(N, K, w.splits, parts, C, ldc, s);
}

}  // namespace

namespace {
// The workspace of a packed route whose operands take `need` bytes, in a call that
// otherwise asks for `plain`.  The size is what tells the two routes apart, so it
// exceeds the plain one, rounded up as that is given out; and a weight takes 6
// bytes, stored or zero, so beyond 4 GiB (26,000 x 26,000 weights) the call keeps to
// its stored entries (0: 65536 x 65536 at 20 % would take 26 GB beside 7 of W).
constexpr size_t kPackedMost = (size_t)4 << 30;
size_t packed_size(size_t need, size_t plain) {
    const size_t n = need > plain + 256 ? need : plain + 256;
    return n <= kPackedMost ? n : 0;
}
}  // namespace

// Where the split product is taken (times in us, fp32 tiles -> split product,
// dense_wgrad).  The packing launch costs 5-6 us, so the batch has to be long
// enough for the faster products to win it back.  F32: 2048 x 2048 x 64 12.1 ->
// 17.1, 2000 x 300 x 128 15.1 -> 17.4, 300 x 784 x 256 24.5 -> 18.5, 4096 x 9216
// x 128 103 -> 79 (with the prox epilogue 128 -> 115; x 64: 86 -> 93).  And
// where an output is small against long operands, packing moves more than the
// products save: 50 x 500 x 16384 42.8 -> 59.5, 128 x 1000 x 20000 74 -> 107, 100
// x 1000 x 3000 33.3 -> 29.4, 300 x 9216 x 1024 114 -> 70.  BF16X3 (whose other
// path does not split a reduction): 2048 x 2048 x 256 17.0 -> 19.6, 2049 x 3001 x
// 333 47 -> 31, 4096 x 4096 x 512 67 -> 60, 50 x 500 x 16384 712 -> 50.
// Rows that are 16-byte aligned let the other kernels load vectors, and outputs
// that fill the chip once let them run without a last partial round (up to 512
// tiles with two BF16X3 workgroups on a CU, 256 tiles with one of fp32): there the
// batch has to be longer.  F32 500 x 8000 x 96 14.0 -> 15.9, x 160 19.4 -> 20.6, x 224
// 24.4 -> 24.6, 2048 x 2048 x 128 16.7 -> 17.3.  BF16X3: x3_unpacked().
namespace {
// The line rises with the tiles to pack for, falls where the last tiles are partly
// empty, which costs the other kernel more, and lies past 512 indices where
// the packed product would be cut into two ranges there.  Other kernel -> packed,
// us: 3072 x 2560 x 512 34.3 -> 36.5, x 608 41.0 -> 40.2; 4096 x 2048 x 320 25.6 -> 30.1; 2600 x 2600 x
// 448 31.7 -> 33.3, x 576 39.9 -> 37.7; 2048 x 2048 x 384 21.5 -> 23.3, x 544 27.6 -> 28.0, x 640 31.4 ->
// 30.1; 1024 x 3072 x 384 20.6 -> 21.7, x 512 25.1 -> 25.1; 1700 x 1700 x 320 20.2 -> 20.8, x 512
// 28.7 -> 26.3; 800 x 2600 x 320 19.9 -> 18.8, x 512 28.2 -> 24.3; 1300 x 1300 x 448 26.2 -> 22.7;
// 1024 x 2048 x 448 22.3 -> 21.9, x 512 24.2 -> 26.0, x 576 26.8 -> 26.9.  768 tiles, 3000 x 4000 x
// 320: 41.5 -> 37.2.  Cards put it apart: 4000 x 2000 x 512 33.4 -> 35.6 on one, 37.3 ->
// 37.2 on another.
bool x3_unpacked(int N, int K, int B, int64_t tiles) {
    if (B % 4 || tiles > 512) return false;
    const bool whole = N % BM == 0 && K % BN == 0;
    if (tiles > 256) return B < (whole ? 600 : 516);
    if (tiles > 200) return B < (whole ? 540 : 416);
    if (tiles > 128) return whole ? B < 450 : tiles > 160 && B < 384;
    return whole && tiles > 112 && B >= 512 && B < 560;
}
}  // namespace
size_t split_wgrad_bytes(int N, int K, int B, int precision) {
    const bool f32 = precision == kPrecF32;
    if ((!f32 && precision != kPrecBF16X3) || N == 0 || K == 0) return 0;
    const double nk = (double)N * K, rows = (double)N + K;
    const int64_t tiles = ceil_div(N, BM) * ceil_div(K, BN);
    if (f32) {
        if (B < (nk >= 4e6 ? 96 : 160)) return 0;
        if (nk < 200 * rows && rows * B > 4e6) return 0;
        if (B % 4 == 0 && tiles > 192 && tiles <= 256 && B < 208) return 0;
    } else if (B < 320 || x3_unpacked(N, K, B, tiles)) {
        return 0;
    }
    if (B > (1 << 22)) return 0;  // 32-bit offsets inside a group
    const int np = f32 ? 3 : 2;
    // (split_plan() makes no more ranges than wgrad_plan())
    const size_t plain = wgrad_workspace_bytes(N, K, B);
    return packed_size((size_t)(packed_bytes(N, B, np) + flag_bytes(N, B) + packed_bytes(K, B, np) + flag_bytes(K, B)) +
                       plain, plain);
}

bool split_wgrad_prox_fused(int N, int K, int B) { return split_plan(N, K, B).splits == 1; }

hipError_t launch_split_wgrad(int N, int K, int B, int precision, const float *dY, int64_t ldy, const float *X,
                              int64_t ldx, float *dW, int64_t ldw, void *ws, hipStream_t s) {
    return precision == kPrecF32
               ? wgrad<3, kEpiStore>(N, K, B, dY, ldy, X, ldx, dW, ldw, prox_epi{}, ws, s)
               : wgrad<2, kEpiStore>(N, K, B, dY, ldy, X, ldx, dW, ldw, prox_epi{}, ws, s);
}

hipError_t launch_split_wgrad_prox(int N, int K, int B, int precision, const float *dY, int64_t ldy, const float *X,
                                   int64_t ldx, float *Z, int64_t ldz, const prox_epi &P, void *ws, hipStream_t s) {
    return precision == kPrecF32 ? wgrad<3, kEpiProx>(N, K, B, dY, ldy, X, ldx, Z, ldz, P, ws, s)
                                 : wgrad<2, kEpiProx>(N, K, B, dY, ldy, X, ldx, Z, ldz, P, ws, s);
}

// gv = dY . X^T on W's pattern: the whole product, its epilogue writing the
// stored entries.  Taken where the modelled time is shorter than the entry-wise
// kernels' (both models in us, fitted to calls on the chip): theirs is nnz * B
// products at 6.6 per ps (dense patterns 12, rows not 16-byte aligned 3.5) or an
// entry's fixed cost, this
// one's the packing, N * K * B products at tile granularity (few tiles: the steps
// of one, 0.55 us each) and the bitmap index.
// Measured at 4096 x 4096 x 512, entry-wise -> whole: 5 % stored 81 -> 105, 10 %
// 135 -> 106, 20 % 259 -> 111, 50 % 369 -> 128; 4096 x 9216 x 1024 at 9 % 693 ->
// 393; 503 x 7856 x 736 at 20 % 143 -> 68, 1738 x 1321 x 531 77 -> 45 (10 % 40 -> 44);
// 1000 x 1000 x 256 at 20 % 22 -> 29, 1024 x 1024 x 1024 43 -> 57; 4096 x 9216 x 64 at 3 % 62 -> 74, 757 x
// 7865 x 51 at 8 % 26 -> 29, 1497 x 11913 x 43 at 5 % 42 -> 53, 569 x 1700 x 32 at 41 % 59 -> 20.
size_t packed_sddmm_bytes(int N, int K, int64_t nnz, int B) {
    if (B < 32 || B > (1 << 22) || N == 0 || K == 0) return 0;
    const double np = (double)ceil_div(N, BM) * BM, kp = (double)ceil_div(K, BN) * BN, n = (double)nnz;
    const double mfma = 12 * np * kp * B / 1.25e9, chain = 0.55 * ceil_div(B, kStep);
    // batches under 256 do not cover a tile's first loads, mask and stores (11 us per 1000 tiles)
    const double tiles = np * kp / (BM * BN), edge = B < 256 ? 11e-3 * tiles * (1 - B / 256.0) : 0;
    const double wide = K > 10240 ? 10 : 0;  // the bitmap index of such rows is made word by word
    const double whole = 24 + 10.0 * ((double)N + K) * B / 5e6 + (mfma > chain ? mfma : chain) + n / 250e3 + edge + wide;
    const double rate = B % 4 ? 3.5e6 : (3 * n > (double)N * K ? 12e6 : 6.6e6);  // products per us
    const double products = n * B / rate, fixed = n / 23e3;
    if (whole > (B < 256 ? 0.92 : 0.88) * (14 + (products > fixed ? products : fixed))) return 0;
    const size_t need = (size_t)(packed_bytes(N, B, 3) + flag_bytes(N, B) + packed_bytes(K, B, 3) + flag_bytes(K, B)) +
                        2 * (size_t)ceil_div(word_counts_bytes(N, K), 256) * 256;
    return packed_size(need, sddmm_workspace_bytes(N, K, nnz, B));
}

hipError_t launch_packed_sddmm(int N, int K, const int *ptr, const int *idx, const float *dY, int64_t ldy,
                               const float *X, int64_t ldx, int B, float *gv, void *ws, hipStream_t s) {
    char *p = static_cast<char *>(ws);
    gemm_args G{};
    G.A = carve_packed(p, N, B, 3);
    G.B = carve_packed(p, K, B, 3);
    unsigned *mask = reinterpret_cast<unsigned *>(p);
    int *pos = reinterpret_cast<int *>(p + ceil_div(word_counts_bytes(N, K), 256) * 256);
    G.a_v4 = ldy % 4 == 0 && aligned16(dY); G.b_v4 = ldx % 4 == 0 && aligned16(X);
    hipError_t e = launch_bitmap(N, K, ptr, idx, mask, pos, s);
    if (e == hipSuccess)
        e = launch_pack<3>(pack_src{dY, ldy, N, G.a_v4, G.A},
                           pack_src{X, ldx, K, G.b_v4, G.B}, B, s);
    if (e != hipSuccess) return e;
    G.M = N; G.Nn = K; G.Kr = B;
    G.a32 = dY; G.lda = ldy; G.b32 = X; G.ldb = ldx;
    G.split_steps = G.A.steps;
    G.C = gv;
    G.P.mask = mask; G.P.pos = pos; G.P.kw = (int)ceil_div(K, 32);
    return launch_tiles<3, kEpiMask, kAccTree>(G, 1, s);
}

// Y = W . X with W's zeros written out: N * K * B products on the matrix cores
// instead of nnz * B on the vector units.  Taken where the modelled time is
// shorter than the sparse kernels' (both in us, fitted to calls on the chip):
// the tiled kernel costs 60 us of planning and tile passes and 1 us per 12 M
// products, the row kernel (under 1.7e8 products, or rows that are not 16-byte
// aligned) 1 us per 4.5 M or 2.7 M; this one packs 6 bytes per weight and 10 per
// activation, multiplies whole tiles and adds split sums.  Measured, sparse ->
// packed: 4096 x 4096 x 512 at 5 % stored 108 -> 105, 10 % 126 -> 107, 20 % 197 ->
// 114, 50 % 316 -> 128; 4096 x 9216 x 1024 at 9 % 357 -> 401 (W^T 299 -> 445);
// 2049 x 3001 x 333 at 30 % 225 -> 59; 2000 x 700 x 1000 at 25 % 66 -> 39.
namespace {
// Ranges of whole 256-index blocks, about 512 workgroups; ranges of a single block
// only for the first 256 of them (a partial sum costs as much as some 200 indices:
// 6544 x 522 x 832 67 -> 53 us whole, 1000 x 4000 x 300 48.5 -> 44.6 with 8 ranges for
// 16, 2048 x 2048 x 512 46.4 -> 43.6; 2000 x 700 x 1000 39.3 -> 41.8.  256 workgroups
// for all: 3000 x 3000 x 700 111 -> 130, 4096 x 4096 x 512 at 10 % 117 -> 126)
wgrad_split spmm_splits(int N, int K, int B) {
    const int64_t tiles = ceil_div(N, BM) * ceil_div(B, BN), kb = ceil_div(K, kPackK);
    int64_t s = tiles >= 384 ? 1 : ceil_div(512, tiles);
    const int64_t two = kb / 2, fill = ceil_div(256, tiles), most = two > fill ? two : fill;
    s = s < most ? s : most;
    s = s < kb ? s : kb;
    const int64_t per = ceil_div(kb, s > 0 ? s : 1);
    return wgrad_split{(int)ceil_div(kb, per), (int)per * kPackK};
}

// The models above are fitted where packing gains most.  At their line they were up to
// 1.6x wrong: the tiled kernel has no such fixed cost on few entries, packing slows
// down beyond 12 M weights (its output leaves the last-level cache), and a product
// without a tiled plan runs the row kernel.  These are fitted to 250 products of 200-
// 12000 rows and columns, batches of 32-1024 and 2-56 % stored, within 15 % (us; the
// packed one 25 % beyond 36 M weights).  The row kernel may also wait for its longest
// row (0.056 us an entry), so unless that is bounded the packed product is kept up
// to 1.1 of its time on even rows.  Sparse kernel, packed: 1978 x 5941 x 256 at 7 % 41, 66;
// 8944 x 3077 x 1024 at 11 % 267, 319; 9027 x 5314 x 512 at 12 % 317, 376; 5128 x 8214 x 256 at 14 % 232,
// 252; 1544 x 383 x 512 at 50 % 27, 32; 2350 x 3453 x 256 at 11 % 42, 58; kept: 6662 x 6879 x 432
// at 33 % 638, 400; 441 x 6309 x 256 at 42 % 166, 38.  (Power-law rows would gain some way
// past that line, 525 x 7183 x 512 at 10 % 117, 61, where even ones take 47: sizes cannot
// tell them apart.)
bool packed_spmm_loses(int N, int K, int64_t nnz, int B, const wgrad_split &w) {
    const double np = (double)ceil_div(N, BM) * BM, bp = (double)ceil_div(B, BN) * BN, nk = (double)N * K;
    const double n = (double)nnz, products = n * B, density = n / nk;
    const double packed = 23.4 + 0.594e-6 * nk + (nk > 12e6 ? 1.88e-6 * (nk - 12e6) : 0) + 1.96e-6 * K * (double)B +
                          4.38e-6 * n + 8e-9 * np * K * bp + (w.splits > 1 ? 0.755e-6 * w.splits * N * (double)B : 0) +
                          (density > 0.2 ? 8 * (density - 0.2) : 0);
    if (B % 4 == 0 && spmm_workspace_bytes(N, K, nnz, B) > 0)  // the tiled kernel
        return packed > (nk > 36e6 ? 0.8 : 1.04) * (36.6 + products / 21.8e6 + 13e-6 * n + 11.7e-3 * K);
    const double rate = B % 4 ? (B % 2 ? 3.6e6 : 4.2e6) : (B > 2 * kWave ? 5.9e6 : (B > kWave ? 3.8e6 : 2.5e6));
    const double chain = 0.056 * n / N, even = 6 + (products / rate > chain ? products / rate : chain);
    return packed > (0.056 * K < even ? 0.95 : 1.1) * even;
}
}  // namespace

size_t packed_spmm_bytes(int N, int K, int64_t nnz, int B) {
    if (N == 0 || K == 0 || B < 32 || K > (1 << 22)) return 0;
    const wgrad_split w = spmm_splits(N, K, B);
    const double np = (double)ceil_div(N, BM) * BM, bp = (double)ceil_div(B, BN) * BN, nk = (double)N * K;
    const double mfma = 12 * np * K * bp / 1.36e9, stream = 6 * nk / 3.5e6;
    const double packed_us = 28 + 0.85 * ((6 * nk + 10.0 * K * B) / 4.8e6 + (mfma > stream ? mfma : stream) +
                                          (w.splits > 1 ? 8.0 * w.splits * N * B / 6.9e6 : 0));
    const double products = (double)nnz * B;
    const double sparse_us = B % 4 ? 5 + products / 2.7e6
                                   : (products < 1.7e8 ? 5 + products / 4.5e6 : 60 + products / 12e6);
    if (packed_us > 0.95 * sparse_us || packed_spmm_loses(N, K, nnz, B, w)) return 0;
    const size_t need = (size_t)(packed_bytes(N, K, 3) + flag_bytes(N, K) + packed_bytes(B, K, 3) + flag_bytes(B, K)) +
                        (w.splits > 1 ? sizeof(float) * (size_t)w.splits * N * B : 0);
    return packed_size(need, spmm_workspace_bytes(N, K, nnz, B));
}

hipError_t launch_packed_spmm(int N, int K, const int *ptr, const int *idx, const float *vals, const float *X,
                              int64_t ldx, int B, float *Y, int64_t ldy, void *ws, hipStream_t s) {
    char *p = static_cast<char *>(ws);
    gemm_args G{};
    G.A = carve_packed(p, N, K, 3);
    G.B = carve_packed(p, B, K, 3);
    dim3 grid((unsigned)(G.A.groups + G.B.groups), (unsigned)G.A.kblocks);
    pack_spmm_kernel<<<grid, 256, 0, s>>>(N, ptr, idx, vals, G.A, X, ldx, K, B, G.B);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const wgrad_split w = spmm_splits(N, K, B);
    G.M = N; G.Nn = B; G.Kr = K;
    G.b32 = X; G.ldb = ldx;
    G.ptr = ptr; G.idx = idx; G.vals = vals;
    G.split_steps = w.chunk / kStep;
    float *parts = reinterpret_cast<float *>(p);
    G.C = w.splits > 1 ? parts : Y;
    G.ldc = w.splits > 1 ? B : ldy;
    e = launch_tiles<3, kEpiSpmm, kAccSmall>(G, w.splits, s);
    if (e != hipSuccess || w.splits == 1) return e;
    return launch_wgrad_reduce(N, B, w.splits, parts, Y, ldy, s);
}

}  // namespace l1csr
