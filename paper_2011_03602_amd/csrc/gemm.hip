// FP32 matrix product on the matrix cores: the GPU routine a recognised host
// matrix-product block is replaced with (function-block offload, Sec. 3.2.2,
// Sec. 4.2.1).
//
// C = A B for row-major FP32 matrices, in two forms; launch_gemm_f32 picks.
//
// Split form (large products): 128 x 128 tiles staged through LDS, each FP32
// value as the exact sum of three bfloat16 parts, multiplied on the bfloat16
// matrix instructions with FP32 accumulation. Direct form (small and narrow
// products): tiles of 16 x 16 to 32 x 32 on the FP32 matrix instructions, K
// shared among a work-group's waves, operands straight from global memory.
//
// Errors against FP64, root mean square over C, as a fraction of those of one FP32
// sum over all of K on the FP32 instructions (K from 64 to 8192): normally
// distributed values 0.26-0.74 for the direct form, which adds up K in several
// partial sums, and 0.23-0.35 for the split form; rows of A that are a softmax of
// 3 times such values 0.26-0.74 and 0.26-0.49; of 20 times such values, where one
// product dominates a sum, 0.77-0.95 and 0.88-1.09. (At K = 32 the direct form's
// sum has one part and the fraction is 1.) A sum of a single product is within
// 0.506 ulp in the split form, 0.5 in the other.
//
// Operand layouts (wave64, lane l): the 32x32x2 FP32 instruction takes
// A[l % 32][l / 32] and B[l / 32][l % 32], the 16x16x4 one A[l % 16][l / 16] and
// B[l / 16][l % 16], the 32x32x16 bfloat16 one eight consecutive k from
// 8 (l / 32) of row (column) l % 32. Accumulator register r holds row
// 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of a 32 x 32 tile, and row
// 4 (l / 16) + r, column l % 16 of a 16 x 16 one.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ofl_internal.hpp"

namespace ofl {

namespace {

constexpr int kXcds = 8;    // accelerator complex dies of an MI355X, each with its own L2
constexpr int kCus = 256;   // compute units of an MI355X

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
// four consecutive floats that start on any element (a global load needs
// 4-byte alignment only)
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

struct GemmArgs {
    int M, N, K;
    const float *A;
    int lda;
    const float *B;
    int ldb;
    float *C;
    int ldc;
};

// Work-groups are dealt round-robin to the eight XCDs. Give each XCD a
// contiguous run of tiles in row-major tile order instead, so that tiles
// sharing rows of A (and neighbouring columns of B) meet in one XCD's L2.
__device__ __forceinline__ int tile_index() {
    const int n = gridDim.x, b = blockIdx.x, per = n / kXcds;
    return b < per * kXcds ? (b % kXcds) * per + b / kXcds : b;
}

// ---- direct form
//
// All KS waves of a work-group compute the same tile of C, each over its own
// chunks of 32 k, dealt in turn (whole 128-byte lines of A's rows), and their
// sums are added in wave order through LDS. A lane loads four consecutive k of
// its A row in one 16-byte load, and the four instructions that use them take k
// in that order (any order of k serves as long as A and B agree), so operands
// need no staging and there is no barrier before the sum: one wave's loads hide
// behind the others' instructions.
//
// Bound by the loads of a tile's operands through L2, or by the latency of one
// wave's share where there are few tiles. Measured, us a launch among repeated ones
// on the same operands, which the last-level cache then holds, against 64- or
// 128-row by 256-column tiles: 8192 x 16 x 4096 22.1 against 566 (135 MB, 6.1 TB/s;
// among calls on changing operands 30.0, 4.6 TB/s), 511 x 333 x 1001 with odd strides
// 9.6 against 183 (calls: 10.7), 1000^3 30.6 against 188, 128 x 128 x 4096 12.2
// against 611, 64 x 4096 x 512 6.3 against 129.
template <int BASE>
struct Mfma;
template <>
struct Mfma<32> {
    typedef floatx16 Acc;
    static constexpr int kRegs = 16, kGroups = 2;  // accumulator registers, k values per instruction
    static __device__ __forceinline__ Acc mul(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
};
template <>
struct Mfma<16> {
    typedef floatx4 Acc;
    static constexpr int kRegs = 4, kGroups = 4;
    static __device__ __forceinline__ Acc mul(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

constexpr int kChunk = 32;

// One wave's sum over chunks first, first + step, ... of K (the last, partial
// chunk among them) of the MT x 1 accumulator tiles at rows m0.., columns n0,
// n0 + COLS, ... Rows and columns beyond the matrix are clamped; their sums are
// never stored.
template <int BASE, int MT, int COLS = 1>
__device__ __forceinline__ void direct_sum(const GemmArgs &g, int m0, int n0, int lane, int first, int step,
                                           typename Mfma<BASE>::Acc (&acc)[MT]) {
    typedef Mfma<BASE> Op;
    constexpr int kStep = 4 * Op::kGroups;  // k per A load
    constexpr int kSteps = kChunk / kStep;
    const int col = lane % BASE, grp = lane / BASE;
    const float *pa[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        pa[i] = g.A + static_cast<size_t>(min(m0 + i * BASE + col, g.M - 1)) * g.lda + 4 * grp;
#pragma unroll
        for (int r = 0; r < Op::kRegs; ++r)
            acc[i][r] = 0.f;
    }
    const float *pb = g.B + min(n0 + COLS * col, g.N - 1);
    struct Chunk {
        float a[MT][kSteps][4];
        float b[kSteps][4];
    };
    auto load = [&](int k0, Chunk &c) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const float4u v = *reinterpret_cast<const float4u *>(pa[i] + k0 + s * kStep);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    c.a[i][s][q] = v[q];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                c.b[s][q] = pb[static_cast<size_t>(k0 + s * kStep + 4 * grp + q) * g.ldb];
        }
    };
    auto mul = [&](const Chunk &c) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    acc[i] = Op::mul(c.a[i][s][q], c.b[s][q], acc[i]);
    };
    // whole chunks, the next one's loads ahead of this one's products
    const int chunks = g.K / kChunk;
    if (first < chunks) {
        Chunk c0;
        load(first * kChunk, c0);
        for (int c = first; c < chunks; c += step) {
            Chunk c1;
            if (c + step < chunks)
                load((c + step) * kChunk, c1);
            __builtin_amdgcn_sched_barrier(0);
            mul(c0);
            c0 = c1;
        }
    }
    // the last K % 32, element by element, by the wave whose turn it is
    if (g.K % kChunk != 0 && first == chunks % step) {
        Chunk c;
        const int k0 = chunks * kChunk;
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = k0 + s * kStep + 4 * grp + q;
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    c.a[i][s][q] = k < g.K ? pa[i][k0 + s * kStep + q] : 0.f;
                c.b[s][q] = k < g.K ? pb[static_cast<size_t>(k) * g.ldb] : 0.f;
            }
        mul(c);
    }
}

template <int BASE, int MT, int KS>
__global__ __launch_bounds__(KS * 64) void gemm_direct_kernel(GemmArgs g, int tiles_n) {
    typedef Mfma<BASE> Op;
    constexpr int TM = BASE * MT;
    __shared__ float sums[KS][TM][BASE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = tile_index();
    const int m0 = t / tiles_n * TM, n0 = t % tiles_n * BASE;
    typename Op::Acc acc[MT];
    direct_sum<BASE, MT>(g, m0, n0, lane, wave, KS, acc);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < Op::kRegs; ++r)
            sums[wave][i * BASE + Op::row(lane, r)][lane % BASE] = acc[i][r];
    __syncthreads();
    for (int e = threadIdx.x; e < TM * BASE; e += KS * 64) {
        const int r = e / BASE, c = e % BASE;
        float v = sums[0][r][c];
#pragma unroll
        for (int w = 1; w < KS; ++w)
            v += sums[w][r][c];
        if (m0 + r < g.M && n0 + c < g.N)
            g.C[static_cast<size_t>(m0 + r) * g.ldc + n0 + c] = v;
    }
}

// ---- split form
//
// x = x0 + x1 + x2 with x0 = bfloat16(x), x1 = bfloat16(x - x0),
// x2 = x - x0 - x1, each rounded to nearest even: FP32's 24 significant bits fit
// three bfloat16 ones of 8, so the sum is exact. Of the nine products of parts all
// but x2 y2 are taken, which is at most 2^-34 of |x y|. Eight bfloat16 instructions
// do the work of eight FP32 ones in half of the matrix cores' time. The instruction
// truncates the lower addends where a product is larger than the sum it joins, so
// x0 y0 has a sum of its own and the other products, 2^-8 of it, another; they are
// added at the end. (Without x1 y2 and x2 y1, which come to 2^-24 of |x y|, and with
// one sum for all, a sum of one product was up to 1.41 ulp off.)
//
// Four waves own a 128 x 128 tile (64 x 64 each). A stage of 32 k is fetched
// into registers, split there and written to LDS in the order the instructions
// read it; each value is split once and feeds 128 rows or columns. A work-group
// has two such groups of four waves on one tile: they take alternate stages, one
// splits while the other multiplies, and their sums are added at the end. With
// one group, two work-groups share a CU instead (at small K, see pick_form).
//
// Measured, us a launch among repeated ones against FP32-instruction tiles of 128 or
// 64 rows by 256 columns: 4096^3 858 against 996 (160 TFLOP/s; 822 among calls on
// changing operands), 8192^3 7000 against 7820, 2048^3 112 against 175, 2340 x 1142
// x 3098 138 against 594. The bfloat16 instructions then run at 1.28 PFLOP/s, above
// the rate a library's large bfloat16 product reaches on this card (1.11), whose
// clock falls below 2 GHz under it. (With six products and one sum: 4096^3 742 among
// calls.)
//
// Range. Operands are split times 2^23 each and the sums stored times 2^-46: then
// every part of every FP32 value, the smallest subnormal one's 2^-149 among them,
// is a normal bfloat16 number (beside a product with a subnormal operand the
// instruction drops up to 7 bits more of a lower addend), and the sums lose nothing
// below the normal range that the results would keep. That leaves no room for
// |x| from 2^104 or |C| from 2^82, so a tile whose first stages hold a value from
// 2^30 splits its operands as they are, and looks out for nonzero values below
// 2^-103, whose parts would be subnormal. A tile that meets one, or whose sums come
// out infinite or NaN, is computed again with the FP32 instructions, straight from
// global memory (4096^3 with every tile so: 3.4 ms): infinite and NaN operands,
// overflow, and operands that mix those magnitudes or grow past the scaled range
// only after the first stages. With operands always split as
// they are and tiles redone below 2^-50, 4096^3 with one operand around 1e-18 took
// 3355 us, since then what other operands take.
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

constexpr int kSplitTile = 128, kSplitK = 32, kParts = 3;
// One part of 32 rows x 32 k in LDS: 8 k of a row are 16 bytes, 32 rows 512, and
// 32 bytes more put the k groups that 16 consecutive lanes write of A (8 bytes
// each, two rows) on distinct banks. B's columns are dealt to the four 32-column
// tiles in turn (tile e: columns 4 c + e), so that a lane's four consecutive
// columns go to the same row of the four tiles, and 16 consecutive lanes write
// both halves of eight rows. No access conflicts (with k groups 640 bytes apart
// and columns in order, a stage's 48 accesses per wave took 330 cycles more).
constexpr int kK8Stride = 512 + 32, kTileStride = 4 * kK8Stride;
constexpr float kSplitScale = 0x1p23f, kSplitLarge = 0x1p30f;
constexpr unsigned kSplitTiny = (127u - 103u) << 24;  // 2^-103, shifted left by one (no sign)

__device__ __forceinline__ void split2(float x, float y, unsigned (&p)[kParts]) {
#pragma unroll
    for (int s = 0; s < kParts; ++s) {
        const bf2 h = __builtin_convertvector(floatx2{x, y}, bf2);
        p[s] = __builtin_bit_cast(unsigned, h);
        if (s + 1 < kParts) {
            x -= __uint_as_float(p[s] << 16);
            y -= __uint_as_float(p[s] & 0xffff0000u);
        }
    }
}

// Orders the work-group's LDS accesses without waiting for its global loads
// (the next stage's are in flight).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int GROUPS>
__global__ __launch_bounds__(256 * GROUPS, 2) void gemm_split_kernel(GemmArgs g, int tiles_n) {
    __shared__ __attribute__((aligned(16))) char lds[GROUPS][2][kParts * 4 * kTileStride];
    __shared__ int redo, large;
    const int tid = threadIdx.x % 256, lane = tid & 63;
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / 256);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char *la = lds[group][0], *lb = lds[group][1];
    const int t = tile_index();
    const int m0 = t / tiles_n * kSplitTile, n0 = t % tiles_n * kSplitTile;
    const bool whole_n = n0 + kSplitTile <= g.N;

    // this thread's share of a stage: A rows ar + 32 i, k ak .. ak+3; B rows
    // bk .. bk+3, columns bn .. bn+3
    const int ar = tid / 8, ak = tid % 8 * 4;
    const int bk = (tid / 64 * 2 + tid % 2) * 4, bn = tid % 64 / 2 * 4;
    const float *pa[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        pa[i] = g.A + static_cast<size_t>(min(m0 + ar + 32 * i, g.M - 1)) * g.lda + ak;
    // past B's last column a thread's load moves back to start at bs; its values
    // move up when they are split (there, so that the loads stay in flight)
    const int bs = min(n0 + bn, max(g.N - 4, 0)), over = n0 + bn - bs;
    float ra[4][4], rb[4][4];
    auto fetch = [&](int k0) {
        if (k0 + kSplitK <= g.K) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4u v = *reinterpret_cast<const float4u *>(pa[i] + k0);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    ra[i][q] = v[q];
            }
            if (g.N >= 4) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4u v =
                        *reinterpret_cast<const float4u *>(g.B + static_cast<size_t>(k0 + bk + q) * g.ldb + bs);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        rb[q][e] = v[e];
                }
                return;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    ra[i][q] = k0 + ak + q < g.K ? pa[i][k0 + q] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                rb[q][e] = k0 + bk + q < g.K
                               ? g.B[static_cast<size_t>(k0 + bk + q) * g.ldb + min(bs + e, g.N - 1)]
                               : 0.f;
    };
    float scale = kSplitScale;
    unsigned tiny = 0xffffffffu;  // smallest nonzero |x| seen, shifted left, less one (zero wraps to the top)
    auto stash = [&] {
        if (scale == 1.f)
#pragma unroll
            for (int t = 0; t < 32; ++t)
                tiny = min(tiny, (__float_as_uint(t < 16 ? ra[t / 4][t % 4] : rb[t / 4 - 4][t % 4]) << 1) - 1u);
        auto put = [&](char *base, int tile, int row, int k, const float *v) {
            unsigned lo[kParts], hi[kParts];
            split2(v[0] * scale, v[1] * scale, lo);
            split2(v[2] * scale, v[3] * scale, hi);
#pragma unroll
            for (int s = 0; s < kParts; ++s)
                *reinterpret_cast<uintx2 *>(base + (s * 4 + tile) * kTileStride + k / 8 * kK8Stride + row * 16 +
                                            k % 8 * 2) = uintx2{lo[s], hi[s]};
        };
        if (!whole_n)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float *v = rb[q];
                if (over & 1)
                    v[0] = v[1], v[1] = v[2], v[2] = v[3];
                if (over & 2)
                    v[0] = v[2], v[1] = v[3];
            }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            put(la, i, ar, ak, ra[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float col[4] = {rb[0][e], rb[1][e], rb[2][e], rb[3][e]};
            put(lb, e, bn / 4, bk, col);
        }
    };
    const int wm = wave / 2 * 2, wn = wave % 2 * 2;  // the wave's first row tile and column tile
    floatx16 acc[2][2], low[2][2];  // sums of a0 b0, and of the other products
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = low[i][j][r] = 0.f;
    const int at = lane / 32 * kK8Stride + lane % 32 * 16;
    auto multiply = [&] {
#pragma unroll
        for (int kb = 0; kb < kSplitK / 16; ++kb) {
            bf8 a[2][kParts], b[2][kParts];
#pragma unroll
            for (int s = 0; s < kParts; ++s)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int off = kb * 2 * kK8Stride + at;
                    a[i][s] = *reinterpret_cast<const bf8 *>(la + (s * 4 + wm + i) * kTileStride + off);
                    b[i][s] = *reinterpret_cast<const bf8 *>(lb + (s * 4 + wn + i) * kTileStride + off);
                }
            // the small products first
#pragma unroll
            for (int sum = kParts; sum >= 0; --sum)
#pragma unroll
                for (int s = max(0, sum - kParts + 1); s <= min(sum, kParts - 1); ++s)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            floatx16 &c = sum > 0 ? low[i][j] : acc[i][j];
                            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][s], b[j][sum - s], c, 0, 0, 0);
                        }
        }
    };
    if (threadIdx.x == 0)
        redo = large = 0;
    const int stages = (g.K + kSplitK - 1) / kSplitK;
    lds_barrier();
    if (group < stages) {
        fetch(group * kSplitK);
        float top = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                top = fmaxf(top, fmaxf(fabsf(ra[i][q]), fabsf(rb[i][q])));
        if (top >= kSplitLarge)
            large = 1;
    }
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(large) != 0)
        scale = 1.f;
    if constexpr (GROUPS == 1) {
        for (int p = 0; p < stages; ++p) {
            stash();
            lds_barrier();
            if (p + 1 < stages)
                fetch((p + 1) * kSplitK);
            __builtin_amdgcn_sched_barrier(0);
            multiply();
            lds_barrier();
        }
    } else {
        // phase p: group p % 2 multiplies stage p while the other writes stage p + 1
        if (group == 0 && stages > 0)
            stash();
        lds_barrier();
        for (int p = 0; p < stages; ++p) {
            if (group == (p & 1)) {
                if (p + 2 < stages)
                    fetch((p + 2) * kSplitK);
                __builtin_amdgcn_sched_barrier(0);
                multiply();
            } else if (p + 1 < stages) {
                stash();
            }
            lds_barrier();
        }
    }

    unsigned top = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] += low[i][j][r];
                top = max(top, __float_as_uint(acc[i][j][r]) & 0x7fffffffu);
            }
    if (tiny < kSplitTiny - 1u || top >= 0x7f800000u)
        redo = 1;
    __syncthreads();  // the stages are read
    // Through LDS, where the groups' sums meet, to rows of C in order: first the
    // even 32-row tiles, then the odd ones.
    constexpr int kHalf = kSplitTile / 2 * kSplitTile;
    float *out = reinterpret_cast<float *>(&lds[0][0][0]);
    static_assert(GROUPS * kHalf * sizeof(float) <= sizeof lds, "the sums fit the stages' place");
    const float unscale = 1.f / (scale * scale);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            *reinterpret_cast<floatx2 *>(out + group * kHalf + (wm * 16 + Mfma<32>::row(lane, r)) * kSplitTile +
                                         4 * (lane % 32) + wn) =
                floatx2{acc[i][0][r] * unscale, acc[i][1][r] * unscale};
        __syncthreads();
        for (int e = threadIdx.x; e < kHalf / 4; e += 256 * GROUPS) {
            float4u v = *reinterpret_cast<const floatx4 *>(out + 4 * e);
            if constexpr (GROUPS == 2)
                v += *reinterpret_cast<const floatx4 *>(out + kHalf + 4 * e);
            const int r = e / (kSplitTile / 4), row = m0 + (r / 32 * 2 + i) * 32 + r % 32;
            const int c = n0 + e % (kSplitTile / 4) * 4;
            if (row < g.M) {
                float *p = g.C + static_cast<size_t>(row) * g.ldc + c;
                if (c + 4 <= g.N)
                    *reinterpret_cast<float4u *>(p) = v;
                else
                    for (int q = 0; c + q < g.N; ++q)
                        p[q] = v[q];
            }
        }
        __syncthreads();
    }
    // (here, where the sums are no longer held in registers)
    if (redo != 0) {
        for (int i = group; i < 2; i += GROUPS)
            for (int j = 0; j < 2; ++j) {
                floatx16 sum[1];
                const int mt = m0 + (wm + i) * 32, c = n0 + 4 * (lane % 32) + wn + j;
                direct_sum<32, 1, 4>(g, mt, n0 + wn + j, lane, 0, 1, sum);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = mt + Mfma<32>::row(lane, r);
                    if (row < g.M && c < g.N)
                        g.C[static_cast<size_t>(row) * g.ldc + c] = sum[0][r];
                }
            }
    }
}

enum class Form { kDirect16, kDirect32x16, kDirect32, kSplit, kSplitShared };

long long tiles(const GemmArgs &g, int tm, int tn) {
    return static_cast<long long>((g.M + tm - 1) / tm) * ((g.N + tn - 1) / tn);
}

// The form with the least estimated time, in microseconds. A direct form's
// rounds of one tile per CU take a fixed cost and a share of K each; a split one's rounds of
// resident tiles (two groups: one per CU, and a part-filled last round is
// faster; one group: two per CU, better at small K, where a tile's fixed cost
// counts) a fixed cost and a share. Fitted to 144 products (M 64..8192, N 8..8192,
// K 32..8192): on those the choice takes 1.01 times the best form's time on average,
// 1.33 at worst (of 4 us).
Form pick_form(const GemmArgs &g) {
    const double k = g.K;
    auto direct = [&](int tm, int tn, double fixed, double share) {
        return 3.0 - fixed + (fixed + k * share) * static_cast<double>((tiles(g, tm, tn) + kCus - 1) / kCus);
    };
    const long long big = tiles(g, kSplitTile, kSplitTile);
    auto rounds = [&](int slots) { return static_cast<double>(big / slots); };
    auto rest = [&](int slots) { return static_cast<double>(big % slots) / slots; };
    const double alone = 5.0 + rounds(2 * kCus) * (4.8 + 0.101 * k) +
                         (rest(2 * kCus) > 0 ? 4.8 + k * (rest(2 * kCus) > 0.5 ? 0.101 : 0.061) : 0.0);
    const double shared =
        5.0 + rounds(kCus) * (4.3 + 0.0556 * k) + (rest(kCus) > 0 ? 4.3 + k * (0.0354 + 0.0142 * rest(kCus)) : 0.0);
    const double us[] = {direct(16, 16, 0.5, 2.7e-3), direct(32, 16, 0.3, 5.2e-3), direct(32, 32, 0.5, 6.9e-3),
                         alone, shared};
    // A launch holds fewer than 2^32 threads; past that the count wraps without an
    // error and most of C is not written. Few rows of 2^28 columns would be past it in
    // 16- or 32-column tiles; kSplit, with two threads per column, always fits.
    const long long threads[] = {1024 * tiles(g, 16, 16), 512 * tiles(g, 32, 16), 512 * tiles(g, 32, 32), 256 * big,
                                 512 * big};
    int best = static_cast<int>(Form::kSplit);
    for (int f = 0; f < 5; ++f)
        if (us[f] < us[best] && threads[f] < (1LL << 32))
            best = f;
    return static_cast<Form>(best);
}

template <int BASE, int MT, int KS>
void run_direct(const GemmArgs &g, hipStream_t s) {
    const int tn = (g.N + BASE - 1) / BASE;
    gemm_direct_kernel<BASE, MT, KS>
        <<<static_cast<unsigned>(tiles(g, BASE * MT, BASE)), KS * 64, 0, s>>>(g, tn);
}

}  // namespace

void launch_gemm_f32(int M, int N, int K, const float *A, int lda, const float *B, int ldb, float *C, int ldc,
                     hipStream_t s) {
    const GemmArgs g{M, N, K, A, lda, B, ldb, C, ldc};
    const int tn = (N + kSplitTile - 1) / kSplitTile;
    const unsigned big = static_cast<unsigned>(tiles(g, kSplitTile, kSplitTile));
    switch (pick_form(g)) {
    case Form::kDirect16:
        run_direct<16, 1, 16>(g, s);
        break;
    case Form::kDirect32x16:
        run_direct<16, 2, 8>(g, s);
        break;
    case Form::kDirect32:
        run_direct<32, 1, 8>(g, s);
        break;
    case Form::kSplit:
        gemm_split_kernel<1><<<big, 256, 0, s>>>(g, tn);
        break;
    case Form::kSplitShared:
        gemm_split_kernel<2><<<big, 512, 0, s>>>(g, tn);
        break;
    }
    hip_check(hipGetLastError(), "gemm kernel launch");
}

}  // namespace ofl
