// The pair sweep: two Jacobi iterations (S, R, C, S, R, C) in one pass over the
// coefficients.
//
// A sweep is bound by its twelve coefficient streams (48 of 56 bytes per point
// in FP32). Here a work-group applies iteration n+1 to a plane one step after
// iteration n, while the plane's coefficients are still on the chip, so they
// come from HBM once for two iterations, p is read and written once, and the
// iterate between the two never leaves the chip. p's new values go to the other
// buffer, which makes both copy-backs exact buffer exchanges (as in the fused
// iteration), and each iteration's residual terms are summed on the way.
//
//  * W waves march along k. At plane m every wave relaxes its points once (step
//    1) and leaves the result u in LDS; after a barrier the work-group relaxes
//    plane m-1 again (step 2) from the u of planes m-2..m. Step 2 needs u one
//    point further out in i and j, so a work-group computes step 1 on a margin
//    that its neighbour computes too; the margin's coefficients are fetched
//    with ordinary loads, from the XCD's L2 where the neighbour's loads left
//    them (work-groups of one XCD are neighbours), the rest non-temporally.
//  * Row form: a wave owns 64*VEC points of one row; rows 0 and W-1 of the
//    work-group are the margin in j, and tiles of long rows overlap by the
//    margin in i. Flat form (batches, and rows that tiles fit badly): the
//    work-group covers 256*W consecutive points of a plane across row ends, the
//    margin is a row and a point at each end, and no lane idles on short rows.
//  * The stencil is kept per plane as rows a, c, b (j-1, j, j+1), d = b - a and
//    the right-minus-left differences of c and d: the corner sums of the sweep
//    are differences of these, so every point gets the sweep's own operations
//    in its own order (results are bitwise the sweep's) with fewer of them, and
//    a window of three planes takes 9*VEC+2 registers per step.
//  * With 4 points per lane the next plane's coefficients travel to LDS
//    directly (16 bytes per lane) while the current plane is computed: they need
//    no registers on the way, of which the coefficients of two planes and two
//    windows leave none. Each slot is refilled as soon as it has been read, so
//    the loads in flight never drain. In bfloat16 a plane is half the bytes, too
//    few in flight for HBM's latency, and LDS holds two planes: the one after
//    the next is fetched too (257x257x513: 245 -> 215 us per pair). Narrower rows
//    fetch without LDS; there several work-groups share a CU and overlap.
//  * The march alternates between two sets of registers for each window's planes
//    and the coefficients, two planes per turn of the loop. Moving them at every
//    plane's end took a third of the instructions: FP32 367 -> 361 us per pair,
//    161x161x321 in one round of work-groups 89.7 -> 84.8, bfloat16 there 78.0 ->
//    70.2 (with the deeper fetch).
//
// Measured at 257x257x513, an iteration as three nests against half a pair:
// FP32 385 -> 181 us, bfloat16-offset 265 -> 108 us (as one fused sweep: 316 and
// 188). A pair moves 1.97 GB of HBM in FP32 (1.86 the least; 5.4 TB/s) and took
// 357 us with its arithmetic left out: the loads bound it, and of the 88% of the
// streaming rate that it reaches the margins' L2 reads and the fill of each
// march are the rest.
#include <algorithm>
#include <type_traits>

#include "pair.hpp"

namespace ofl {
namespace {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
#define OFL_GLOBAL __attribute__((address_space(1)))
#define OFL_LDS __attribute__((address_space(3)))

// A lane's VEC consecutive points in FP32 (F) and bfloat16 (H).
template <int VEC>
struct VecOf;
template <>
struct VecOf<1> {
    typedef float F;
    typedef uint16_t H;
};
template <>
struct VecOf<2> {
    typedef f2 F;
    typedef unsigned H;
};
template <>
struct VecOf<4> {
    typedef f4 F;
    typedef u2 H;
};

template <int VEC>
__device__ __forceinline__ void unpack(typename VecOf<VEC>::F x, float (&v)[VEC]) {
    if constexpr (VEC == 1)
        v[0] = x;
    else
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            v[e] = x[e];
}

template <int VEC>
__device__ __forceinline__ typename VecOf<VEC>::F pack(const float (&v)[VEC]) {
    if constexpr (VEC == 1) {
        return v[0];
    } else {
        typename VecOf<VEC>::F x;
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            x[e] = v[e];
        return x;
    }
}

// A wave-uniform address kept in scalar registers, and a lane offset whose
// widening to 64 bits stays beside its use: the access then adds the two itself
// (hoisted out of the loop, every address would be a per-lane 64-bit sum).
__device__ __forceinline__ const OFL_GLOBAL char *scalar(const void *p) {
    const OFL_GLOBAL char *q = (const OFL_GLOBAL char *)p;
    asm("" : "+s"(q));
    return q;
}
__device__ __forceinline__ unsigned here(unsigned x) {
    asm("" : "+v"(x));
    return x;
}
template <class T>
__device__ __forceinline__ const OFL_GLOBAL T *at(const void *base, unsigned lane_bytes) {
    return (const OFL_GLOBAL T *)(scalar(base) + here(lane_bytes));
}

// The twelve coefficients of a lane's points as stored: FP32, or bfloat16
// decoded where they are used (the sweep's decode: bias + widened value).
template <int VEC, bool BF16>
struct Coefs {
    typedef typename std::conditional<BF16, typename VecOf<VEC>::H, typename VecOf<VEC>::F>::type T;
    T x[kNCoef];

    __device__ __forceinline__ float get(const GridView &g, int n, int e) const {
        if constexpr (!BF16) {
            if constexpr (VEC == 1)
                return x[n];
            else
                return x[n][e];
        } else {
            unsigned u;
            if constexpr (VEC == 4)
                u = x[n][e / 2];
            else
                u = x[n];
            return g.bias[n] + __uint_as_float((e & 1) ? (u & 0xffff0000u) : (u << 16));
        }
    }
};

// Lane l receives lane l-1's (l+1's) value, lane 0 (63) `edge`.
__device__ __forceinline__ float from_left(float v, float edge) {
    return __uint_as_float(
        __builtin_amdgcn_update_dpp(__float_as_uint(edge), __float_as_uint(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_right(float v, float edge) {
    return __uint_as_float(
        __builtin_amdgcn_update_dpp(__float_as_uint(edge), __float_as_uint(v), 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane));
}

// Values beside a wave's points in rows a, c, b: left of lane 0, right of lane 63.
struct Edges {
    float la, lc, lb, ra, rc, rb;
};

// What one plane contributes to a point's stencil: rows j-1, j, j+1 (a, c, b),
// d = b - a, the right-minus-left differences of c (dc) and of d (dd), and c's
// neighbours across the lane's ends.
template <int VEC>
struct Plane {
    float a[VEC], c[VEC], b[VEC], d[VEC], dc[VEC], dd[VEC];
    float l, r;

    __device__ __forceinline__ void derive(const Edges &h) {
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            d[e] = b[e] - a[e];
        l = from_left(c[VEC - 1], h.lc);
        r = from_right(c[0], h.rc);
        const float dl = from_left(d[VEC - 1], h.lb - h.la);
        const float dr = from_right(d[0], h.rb - h.ra);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            dc[e] = (e < VEC - 1 ? c[e + 1] : r) - (e > 0 ? c[e - 1] : l);
            dd[e] = (e < VEC - 1 ? d[e + 1] : dr) - (e > 0 ? d[e - 1] : dl);
        }
    }
};

// What is still needed of plane k-1 when plane k is updated.
template <int VEC>
struct Behind {
    float c[VEC], d[VEC], dc[VEC];
    __device__ __forceinline__ void keep(const Plane<VEC> &p) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            c[e] = p.c[e];
            d[e] = p.d[e];
            dc[e] = p.dc[e];
        }
    }
};

// The sweep's update of plane k (m) between planes k-1 (z) and k+1 (n),
// operation for operation in the sweep's order.
template <int VEC, bool BF16>
__device__ __forceinline__ void relax(const GridView &g, const Behind<VEC> &z, const Plane<VEC> &m,
                                      const Plane<VEC> &n, const Coefs<VEC, BF16> &C, float omega,
                                      float (&out)[VEC]) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const float rt = e < VEC - 1 ? m.c[e + 1] : m.r;
        const float lf = e > 0 ? m.c[e - 1] : m.l;
        const float centre = m.c[e];
        float s0 = C.get(g, 0, e) * rt;
        s0 = fmaf(C.get(g, 1, e), m.b[e], s0);
        s0 = fmaf(C.get(g, 2, e), n.c[e], s0);
        s0 = fmaf(C.get(g, 4, e), m.dd[e], s0);
        s0 = fmaf(C.get(g, 5, e), n.d[e] - z.d[e], s0);
        s0 = fmaf(C.get(g, 6, e), n.dc[e] - z.dc[e], s0);
        s0 = fmaf(C.get(g, 7, e), lf, s0);
        s0 = fmaf(C.get(g, 8, e), m.a[e], s0);
        s0 = fmaf(C.get(g, 9, e), z.c[e], s0);
        s0 += C.get(g, 11, e);
        const float ss = fmaf(C.get(g, 3, e), s0, -centre) * C.get(g, 10, e);
        out[e] = fmaf(omega, ss, centre);
    }
}

// Orders this work-group's LDS accesses across the barrier without waiting for
// its global loads (which __syncthreads would, and the coefficients of the next
// plane are meant to stay in flight).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// XCD x (work-group id % 8) takes one contiguous range of n items.
__device__ __forceinline__ int xcd_range(int bid, int n) {
    const int xcd = bid % 8, per = n / 8, rem = n % 8;
    return xcd * per + min(xcd, rem) + bid / 8;
}

// Fixed-order sum of x[0..n) by a whole work-group of W waves; valid on thread 0.
template <int W>
__device__ __forceinline__ double group_sum(const double *x, long long n, double *wsum) {
    double v = 0.0;
    for (long long t = threadIdx.x; t < n; t += W * kWave)
        v += x[t];
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1)
        v += __shfl_xor(v, d, kWave);
    __syncthreads();  // wsum may still be read by the caller's last call
    if ((threadIdx.x & (kWave - 1)) == 0)
        wsum[threadIdx.x / kWave] = v;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < W; ++q)
        t += wsum[q];
    return t;
}

// LDS of a work-group.
template <int VEC, bool BF16, int W>
struct Shared {
    static constexpr bool kDma = VEC == 4;
    static constexpr int kDepth = kDma && BF16 ? 2 : 1;  // planes of coefficients fetched ahead
    typename VecOf<VEC>::F u[2][W * kWave];  // step 1's planes m and m-1
    double wsum[2][W];
    // what the waves fetch ahead: the next planes' coefficients, and the rows
    // a, c, b of the plane after it with the values beside them
    typename Coefs<VEC, BF16>::T next[kDepth][kDma ? W : 1][kDma ? kNCoef : 1][kWave];
    typename VecOf<VEC>::F rows[kDma ? W : 1][kDma ? 3 : 1][kWave];
    float beside[kDma ? W : 1][kWave];
};

// One work-group's march: planes [m0, m1) of tile (ts, j0) in row form (points
// from ts, rows j0-1..j0+W-2) or of the flat range from f0. own_lo, own_hi
// bound the points it stores: i in row form, offsets in the plane in flat form.
// part[0] and part[stride] receive its two residual sums.
template <int VEC, bool BF16, int W, bool FLAT>
__device__ __forceinline__ void pair_march(const GridView &g, Shared<VEC, BF16, W> &sh, int ts, int j0, int own_lo,
                                           int own_hi, int m0, int m1, float omega, double *part,
                                           long long stride) {
    typedef typename VecOf<VEC>::F F;
    typedef Coefs<VEC, BF16> C12;
    constexpr bool kDma = Shared<VEC, BF16, W>::kDma;
    constexpr int kDepth = Shared<VEC, BF16, W>::kDepth;
    constexpr int S = kWave * VEC;
    constexpr int kEb = BF16 ? 2 : 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int I = g.I, pitch = g.pitch;

    // The lane's points: i0.. of row j; its loads at `pos` elements from the
    // (wave-uniform) line starts la, lc, lb of rows j-1, j, j+1 in p. Positions
    // outside the arrays are clamped; what is loaded there is never stored.
    // Flat form: a point's place in the coefficient planes, whose rows may have a
    // pitch of their own, for a load of n points.
    auto coef_at = [&](int f, int n) {
        return g.cpitch == pitch ? f : f / pitch * g.cpitch + min(f % pitch, g.cpitch - n);
    };
    int i0, j, pos, cpos;
    long long la, lc, lb, cline;
    bool row_in, row_out, own, shared_rows;
    if constexpr (FLAT) {
        const int last = pitch * g.J - VEC;
        const int f = ts + wave * S + lane * VEC;
        pos = min(max(f, 0), last);
        j = pos / pitch;
        i0 = pos - j * pitch;
        cpos = coef_at(pos, VEC);
        lc = cline = 0;
        la = -static_cast<long long>(pitch);
        lb = pitch;
        row_in = f == pos && j >= 1 && j <= g.J - 2;
        own = f == pos && f >= own_lo && f < own_hi;
        row_out = row_in;
        shared_rows = ts + wave * S < own_lo + pitch || ts + (wave + 1) * S > own_hi - pitch;
    } else {
        j = j0 - 1 + wave;
        i0 = ts + lane * VEC;
        pos = pair_row_at(i0, I, VEC);
        cpos = pair_coef_at(pos, g.cpitch, VEC);
        la = static_cast<long long>(min(max(j - 1, 0), g.J - 1)) * pitch;
        lc = static_cast<long long>(min(j, g.J - 1)) * pitch;
        lb = static_cast<long long>(min(j + 1, g.J - 1)) * pitch;
        cline = static_cast<long long>(min(j, g.J - 1)) * g.cpitch;
        row_in = j >= 1 && j <= g.J - 2;
        row_out = row_in && wave >= 1 && wave <= W - 2;
        own = i0 == pos && i0 >= own_lo && i0 < own_hi;
        shared_rows = wave <= 1 || wave >= W - 2;
    }
    bool in[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        in[e] = row_in && i0 + e >= 1 && i0 + e <= I - 2;
    const unsigned cb = static_cast<unsigned>(cpos) * kEb, pb = static_cast<unsigned>(pos) * 4;
    // flat form: rows j-1 and j+1 of a lane are clamped on their own
    const unsigned pa4 = FLAT ? static_cast<unsigned>(max(pos - pitch, 0)) * 4 : pb;
    const unsigned pb4 = FLAT ? static_cast<unsigned>(min(pos + pitch, pitch * g.J - VEC)) * 4 : pb;
    // The six values beside the wave's points, fetched by lanes 0..5 (a, c, b:
    // left, then right). Row form needs only the right ones, and those only
    // where the row's last point is the first one past the tile.
    const bool edge = FLAT || ts + S == I - 1;
    unsigned eb;
    if constexpr (FLAT) {
        const int f = ts + wave * S + (lane % 3 - 1) * pitch + (lane < 3 ? -1 : S);
        eb = static_cast<unsigned>(min(max(f, 0), pitch * g.J - 1)) * 4;
    } else {
        const long long line = lane % 3 == 0 ? la : (lane % 3 == 1 ? lc : lb);
        eb = static_cast<unsigned>(line + min(ts + S, pitch - 1)) * 4;
    }
    auto spread = [&](float v) {
        Edges h;
        h.la = FLAT ? lane_value(v, 0) : 0.f;
        h.lc = FLAT ? lane_value(v, 1) : 0.f;
        h.lb = FLAT ? lane_value(v, 2) : 0.f;
        h.ra = lane_value(v, 3);
        h.rc = lane_value(v, 4);
        h.rb = lane_value(v, 5);
        return h;
    };

    struct Rows {
        F a, c, b;
        float h;
    };
    auto plane_base = [&](int k) { return g.p + min(max(k, 0), g.K - 1) * g.plane; };
    auto load_rows = [&](int k) {
        const float *q = plane_base(k);
        Rows r;
        r.a = *at<F>(FLAT ? q : q + la, pa4);
        r.c = *at<F>(FLAT ? q : q + lc, pb);
        r.b = *at<F>(FLAT ? q : q + lb, pb4);
        r.h = edge ? *at<float>(q, eb) : 0.f;
        return r;
    };
    // the same through LDS, four loads
    const int wd = kDma ? wave : 0;
    auto fetch_rows = [&](int k) {
        const float *q = plane_base(k);
        auto one = [&](const float *base, unsigned off, int t) {
            __builtin_amdgcn_global_load_lds((OFL_GLOBAL void *)at<char>(base, off),
                                             (OFL_LDS void *)&sh.rows[wd][kDma ? t : 0][0], 16, 0, 0);
        };
        one(FLAT ? q : q + la, pa4, 0);
        one(FLAT ? q : q + lc, pb, 1);
        one(FLAT ? q : q + lb, pb4, 2);
        __builtin_amdgcn_global_load_lds((OFL_GLOBAL void *)at<char>(q, eb), (OFL_LDS void *)&sh.beside[wd][0], 4, 0,
                                         0);
    };
    auto take_rows = [&] {
        Rows r;
        r.a = sh.rows[wd][0][lane];
        r.c = sh.rows[wd][kDma ? 1 : 0][lane];
        r.b = sh.rows[wd][kDma ? 2 : 0][lane];
        r.h = sh.beside[wd][lane];
        return r;
    };
    auto plane_of = [&](const Rows &r, Plane<VEC> &n) {
        unpack<VEC>(r.a, n.a);
        unpack<VEC>(r.c, n.c);
        unpack<VEC>(r.b, n.b);
        n.derive(spread(r.h));
    };
    // whether any point of the wave is relaxed (wave-uniform)
    const bool active = FLAT || row_in;
    auto coef_base = [&](int n, int k) {
        return static_cast<const char *>(g.coef[n]) + (k * g.cplane + cline) * kEb;
    };

    // Coefficients to LDS: FP32, one load per coefficient; bfloat16, one load
    // for two (half a wave's 16-byte loads cover its 256 points).
    unsigned db = cb;
    if constexpr (BF16) {
        const int at8 = (lane & 31) * 8;
        db = 2u * static_cast<unsigned>(FLAT ? coef_at(min(max(ts + wave * S + at8, 0), pitch * g.J - 8), 8)
                                             : pair_coef_at(ts + at8, g.cpitch, 8));
    }
    auto dma = [&](int t, int k, int slot, auto nt) {
        constexpr int kAux = decltype(nt)::value ? 2 : 0;
        auto *dst = (OFL_LDS void *)&sh.next[slot][wd][kDma ? t : 0][0];
        if constexpr (BF16) {
            const char *b0 = coef_base(t, k), *b1 = coef_base(t + 1, k);
            __builtin_amdgcn_global_load_lds((OFL_GLOBAL void *)((lane < 32 ? b0 : b1) + db), dst, 16, 0, kAux);
        } else {
            __builtin_amdgcn_global_load_lds((OFL_GLOBAL void *)at<char>(coef_base(t, k), db), dst, 16, 0, kAux);
        }
    };
    constexpr int kPer = BF16 ? 2 : 1;     // coefficients per load
    constexpr int kGroup = BF16 ? 4 : 3;   // coefficients per refill step
    auto refill = [&](int t0, int k, int slot) {
        if (shared_rows) {
#pragma unroll
            for (int t = t0; t < t0 + kGroup; t += kPer)
                dma(t, k, slot, std::false_type{});
        } else {
#pragma unroll
            for (int t = t0; t < t0 + kGroup; t += kPer)
                dma(t, k, slot, std::true_type{});
        }
    };
    auto take = [&](C12 &c, int t0, int n, int slot) {
#pragma unroll
        for (int t = t0; t < t0 + n; ++t)
            c.x[t] = sh.next[slot][wd][kDma ? t : 0][lane];
    };

    // Alternating register sets take an odd number of planes, the last of which
    // is peeled: an even march starts one plane early, whose results nothing
    // reads. Narrower forms hide the moves behind their second work-group.
    constexpr bool kAlternate = VEC == 4;
    const int start = m0 - 1 - (kAlternate ? (m1 - m0 + 1) & 1 : 0);
    Plane<VEC> p1[2], p2[2];
    Behind<VEC> z1, z2;
    Edges hm = {};
    {
        plane_of(load_rows(start - 1), p1[0]);
        z1.keep(p1[0]);
        const Rows r = load_rows(start);
        plane_of(r, p1[0]);
        hm = spread(r.h);
    }
    Rows nr;
    if constexpr (kDma) {
        auto coefs = [&](int m) {
#pragma unroll
            for (int t = 0; t < kNCoef; t += kGroup)
                refill(t, min(max(m, 1), g.K - 2), (m - start) % kDepth);
            __builtin_amdgcn_sched_barrier(0);
        };
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kDepth == 2)
            coefs(start);
        fetch_rows(start + 1);
        __builtin_amdgcn_sched_barrier(0);
        coefs(start + kDepth - 1);
    } else {
        nr = load_rows(start + 1);
    }

    C12 D[2];  // a plane's coefficients, kept for its second step
    double r1 = 0.0, r2 = 0.0;
    float o[VEC];
    auto store = [&](int k) {
        if (row_out && own)
            __builtin_nontemporal_store(pack<VEC>(o), (OFL_GLOBAL F *)at<F>(g.wrk2 + k * g.plane + (FLAT ? 0 : lc), pb));
    };
    auto step = [&](int m, auto parity, auto last_plane) {
        constexpr bool kLast = decltype(last_plane)::value;
        constexpr int kThis = decltype(parity)::value, kNext = kThis ^ 1;
        C12 &C = D[kThis];
        Plane<VEC> &c = p1[kThis], &n = p1[kNext];
        Rows r;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kDma) {
            // In flight, oldest first (a store among them only makes a wait
            // stricter): FP32, the next plane's rows (4 loads), this plane's
            // coefficients; bfloat16, this plane's coefficients, the rows, the
            // next plane's coefficients.
            constexpr int kLoads = kNCoef / kPer, kStep = kGroup / kPer;
            __builtin_amdgcn_s_waitcnt(0x0f70 | (kLast && kDepth == 2 ? 0 : kLoads));  // vmcnt
            r = take_rows();
            if constexpr (kDepth == 2)
                take(C, 0, kNCoef, kThis);
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): read before it is overwritten
            __builtin_amdgcn_sched_barrier(0);
            if (m > m0 + 1)
                store(m - 2);
            if constexpr (!kLast) {
                fetch_rows(m + 2);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (kDepth == 2) {
                    if (m + 2 <= m1)
#pragma unroll
                        for (int t = 0; t < kNCoef; t += kGroup)
                            refill(t, min(m + 2, g.K - 2), kThis);
                } else {
                    // What has landed is read and its place refilled before the
                    // next is waited for, so that always kLoads - kStep + 4 newer
                    // loads follow the awaited ones.
                    const int k = min(m + 1, g.K - 2);
#pragma unroll
                    for (int t = 0; t < kNCoef; t += kGroup) {
                        __builtin_amdgcn_s_waitcnt(0x0f70 | (kLoads - kStep + 4));
                        take(C, t, kGroup, 0);
                        __builtin_amdgcn_s_waitcnt(0xc07f);
                        __builtin_amdgcn_sched_barrier(0);
                        refill(t, k, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            } else if constexpr (kDepth == 1) {
                __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
                take(C, 0, kNCoef, 0);
            }
        } else {
            r = nr;
            if (m > m0 + 1)
                store(m - 2);
            if constexpr (!kLast)
                nr = load_rows(m + 2);
            if (active) {
                const int k = min(max(m, 1), g.K - 2);
#pragma unroll
                for (int t = 0; t < kNCoef; ++t) {
                    const OFL_GLOBAL auto *q = at<typename C12::T>(coef_base(t, k), cb);
                    C.x[t] = shared_rows ? *q : __builtin_nontemporal_load(q);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        plane_of(r, n);
        float u[VEC];
        if (active && m >= 1 && m <= g.K - 2) {
            relax(g, z1, c, n, C, omega, u);
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                u[e] = in[e] ? u[e] : c.c[e];
            if (row_out && own && m >= m0 && m < m1) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const double x = static_cast<double>(u[e] - c.c[e]);
                    r1 = fma(x, x, r1);
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                u[e] = c.c[e];
        }
        z1.keep(c);
        F *um = sh.u[m & 1];
        const int at_u = wave * kWave + lane;
        um[at_u] = pack<VEC>(u);
        lds_barrier();
        if (FLAT || row_out) {
            Plane<VEC> &c2 = p2[kThis], &n2 = p2[kNext];
            if constexpr (FLAT) {
                const int step = pitch / VEC, end = W * kWave - 1;
                unpack<VEC>(um[max(at_u - step, 0)], n2.a);
                unpack<VEC>(um[min(at_u + step, end)], n2.b);
                const float *uf = reinterpret_cast<const float *>(um);
                const int f = wave * S + (lane % 3 - 1) * pitch + (lane < 3 ? -1 : S);
                hm = spread(uf[min(max(f, 0), W * S - 1)]);
            } else {
                unpack<VEC>(um[at_u - kWave], n2.a);
                unpack<VEC>(um[at_u + kWave], n2.b);
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                n2.c[e] = u[e];
            n2.derive(hm);
            if (m > m0) {
                relax(g, z2, c2, n2, D[kNext], omega, o);
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    o[e] = in[e] ? o[e] : c2.c[e];
                if (row_out && own) {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        const double x = static_cast<double>(o[e] - c2.c[e]);
                        r2 = fma(x, x, r2);
                    }
                }
            }
            z2.keep(c2);
        }
        // step 2's plane m+1 lies beside the boundary column of p's plane m+1
        if constexpr (!FLAT)
            hm = spread(r.h);
    };
    constexpr std::integral_constant<int, 0> kEven{};
    constexpr std::integral_constant<int, 1> kOdd{};
    if constexpr (kAlternate) {
        for (int m = start; m < m1; m += 2) {
            step(m, kEven, std::false_type{});
            step(m + 1, kOdd, std::false_type{});
        }
    } else {
        for (int m = start; m < m1; ++m) {
            step(m, kEven, std::false_type{});
            p1[0] = p1[1];
            p2[0] = p2[1];
            D[1] = D[0];
        }
    }
    step(m1, kEven, std::true_type{});
    store(m1 - 1);
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        r1 += __shfl_xor(r1, d, kWave);
        r2 += __shfl_xor(r2, d, kWave);
    }
    if (lane == 0) {
        sh.wsum[0][wave] = r1;
        sh.wsum[1][wave] = r2;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double t = 0.0;
        for (int q = 0; q < W; ++q)
            t += sh.wsum[threadIdx.x][q];
        part[threadIdx.x * stride] = t;
    }
}

// One grid. parts: the work-groups' sums of the first iteration, then of the
// second. The last work-group of the launch instead turns the previous pair's
// sums (prev, may be null) into gosa, iteration by iteration.
template <int VEC, bool BF16, int W>
__global__ __launch_bounds__(W *kWave, VEC == 4 ? 1 : 4) void pair_kernel(
    GridView g, PairShape s, float omega, double *parts, const double *prev) {
    constexpr int S = kWave * VEC;
    __shared__ Shared<VEC, BF16, W> sh;
    const int blocks = s.nti * s.njt * s.nkc;
    if (static_cast<int>(blockIdx.x) == blocks) {
        if (prev)
            for (int q = 0; q < 2; ++q) {
                const double t = group_sum<W>(prev + q * blocks, blocks, sh.wsum[0]);
                if (threadIdx.x == 0)
                    *g.gosa = t / (static_cast<double>(omega) * static_cast<double>(omega));
            }
        return;
    }
    const int L = xcd_range(blockIdx.x, blocks);
    const int it = L % s.nti;
    const int jt = (L / s.nti) % s.njt;
    const int kc = L / (s.nti * s.njt);
    const int ts = it * (S - 2 * pair_margin(VEC));
    const int m0 = 1 + kc * s.chunk;
    pair_march<VEC, BF16, W, false>(g, sh, ts, 1 + jt * (W - 2), it == 0 ? 0 : ts + pair_margin(VEC),
                                    it == s.nti - 1 ? g.pitch : ts + S - pair_margin(VEC), m0,
                                    min(m0 + s.chunk, g.K - 1), omega, parts + blockIdx.x, blocks);
}

// One grid in flat form: s.nti segments of a plane, s.nkc chunks.
template <bool BF16, int W>
__global__ __launch_bounds__(W *kWave) void pair_flat_kernel(GridView g, PairShape s, float omega, double *parts,
                                                             const double *prev) {
    __shared__ Shared<4, BF16, W> sh;
    const int blocks = s.nti * s.nkc;
    if (static_cast<int>(blockIdx.x) == blocks) {
        if (prev)
            for (int q = 0; q < 2; ++q) {
                const double t = group_sum<W>(prev + q * blocks, blocks, sh.wsum[0]);
                if (threadIdx.x == 0)
                    *g.gosa = t / (static_cast<double>(omega) * static_cast<double>(omega));
            }
        return;
    }
    const int L = xcd_range(blockIdx.x, blocks);
    const int own = pair_flat_own(g.pitch, W), first = pair_flat_first(g.pitch) + L % s.nti * own;
    const int m0 = 1 + L / s.nti * s.chunk;
    pair_march<4, BF16, W, true>(g, sh, first - pair_flat_margin(g.pitch), 0, first, first + own, m0,
                                 min(m0 + s.chunk, g.K - 1), omega, parts + blockIdx.x, blocks);
}

template <int W>
__global__ __launch_bounds__(W *kWave) void pair_fold_kernel(const double *parts, int n, double omega, double *gosa) {
    __shared__ double wsum[W];
    for (int q = 0; q < 2; ++q) {
        const double t = group_sum<W>(parts + static_cast<long long>(q) * n, n, wsum);
        if (threadIdx.x == 0)
            *gosa = t / (omega * omega);
    }
}

// Many grids in flat form, one item per work-group. parts: two sums per item;
// range[b], range[b+1]: the items of grid b. The last ngrids work-groups turn
// the previous pair's sums (prev, may be null) into each grid's gosa.
template <bool BF16, int W>
__global__ __launch_bounds__(W *kWave) void pair_batch_kernel(const GridView *__restrict__ views,
                                                              const PairItem *__restrict__ items, int nitems,
                                                              const int *__restrict__ range, float omega,
                                                              double *parts, const double *prev) {
    __shared__ Shared<4, BF16, W> sh;
    if (static_cast<int>(blockIdx.x) >= nitems) {
        const int b = blockIdx.x - nitems;
        if (prev)
            for (int q = 0; q < 2; ++q) {
                const double t = group_sum<W>(prev + static_cast<long long>(q) * nitems + range[b],
                                              range[b + 1] - range[b], sh.wsum[0]);
                if (threadIdx.x == 0)
                    *views[b].gosa = t / (static_cast<double>(omega) * static_cast<double>(omega));
            }
        return;
    }
    const int w = xcd_range(blockIdx.x, nitems);
    const PairItem item = items[w];
    const GridView g = views[item.grid];
    const int h = pair_flat_margin(g.pitch);
    pair_march<4, BF16, W, true>(g, sh, item.first - h, 0, item.first, item.first + pair_flat_own(g.pitch, W), item.m0,
                                 item.m1, omega, parts + w, nitems);
}

template <int W>
__global__ __launch_bounds__(W *kWave) void pair_batch_fold_kernel(const GridView *__restrict__ views,
                                                                   const double *__restrict__ parts, int nitems,
                                                                   const int *__restrict__ range, double omega) {
    __shared__ double wsum[W];
    const int b = blockIdx.x;
    for (int q = 0; q < 2; ++q) {
        const double t = group_sum<W>(parts + static_cast<long long>(q) * nitems + range[b], range[b + 1] - range[b],
                                      wsum);
        if (threadIdx.x == 0)
            *views[b].gosa = t / (omega * omega);
    }
}

template <int VEC, bool BF16, int W>
void go(const GridView &g, const PairShape &s, float omega, double *parts, const double *prev, hipStream_t st) {
    pair_kernel<VEC, BF16, W><<<s.blocks() + 1, W * kWave, 0, st>>>(g, s, omega, parts, prev);
}

template <int VEC, int W>
void by_format(const GridView &g, int bf16, const PairShape &s, float omega, double *parts, const double *prev,
               hipStream_t st) {
    if (bf16)
        go<VEC, true, W>(g, s, omega, parts, prev, st);
    else
        go<VEC, false, W>(g, s, omega, parts, prev, st);
}

}  // namespace

void launch_pair(const GridView &g, int bf16, const PairShape &s, float omega, double *parts, const double *prev,
                 hipStream_t st) {
    if (!s.flat && !pair_row_form(s.vec, bf16 ? 2 : 4, g.cpitch))
        fail(OFL_EINVAL, "pair sweep: coefficient rows that 16-byte loads do not divide");
    if (s.flat && s.vec == 4 && s.waves == kPairBatchWaves && s.njt == 1) {
        if (bf16)
            pair_flat_kernel<true, kPairBatchWaves>
                <<<s.blocks() + 1, kPairBatchWaves * kWave, 0, st>>>(g, s, omega, parts, prev);
        else
            pair_flat_kernel<false, kPairBatchWaves>
                <<<s.blocks() + 1, kPairBatchWaves * kWave, 0, st>>>(g, s, omega, parts, prev);
    } else if (s.flat)
        fail(OFL_EINVAL, "pair sweep: no such flat shape");
    else if (s.vec == 4 && s.waves == 8)
        by_format<4, 8>(g, bf16, s, omega, parts, prev, st);
    else if (s.vec == 4 && s.waves == 7)
        by_format<4, 7>(g, bf16, s, omega, parts, prev, st);
    else if (s.vec == 2 && s.waves == 8)
        by_format<2, 8>(g, bf16, s, omega, parts, prev, st);
    else if (s.vec == 1 && s.waves == 8)
        by_format<1, 8>(g, bf16, s, omega, parts, prev, st);
    else
        fail(OFL_EINVAL, "pair sweep: no such shape");
    hip_check(hipGetLastError(), "pair sweep launch");
}

void launch_pair_batch(const GridView *views, const PairItem *items, int nitems, const int *range, int ngrids, int bf16,
                       float omega, double *parts, const double *prev, hipStream_t st) {
    const int blocks = nitems + ngrids;
    if (bf16)
        pair_batch_kernel<true, kPairBatchWaves>
            <<<blocks, kPairBatchWaves * kWave, 0, st>>>(views, items, nitems, range, omega, parts, prev);
    else
        pair_batch_kernel<false, kPairBatchWaves>
            <<<blocks, kPairBatchWaves * kWave, 0, st>>>(views, items, nitems, range, omega, parts, prev);
    hip_check(hipGetLastError(), "batched pair sweep launch");
}

void launch_pair_batch_fold(const GridView *views, const double *parts, int nitems, const int *range, int ngrids,
                            float omega, hipStream_t st) {
    pair_batch_fold_kernel<8><<<ngrids, 8 * kWave, 0, st>>>(views, parts, nitems, range, static_cast<double>(omega));
    hip_check(hipGetLastError(), "batched pair sweep residual launch");
}

void launch_pair_fold(const double *parts, const PairShape &s, float omega, double *gosa, hipStream_t st) {
    pair_fold_kernel<8><<<1, 8 * kWave, 0, st>>>(parts, s.blocks(), static_cast<double>(omega), gosa);
    hip_check(hipGetLastError(), "pair sweep residual launch");
}

}  // namespace ofl
