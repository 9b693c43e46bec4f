// V-Sample / V-Sample-No-Adjust (Alg. 3) for gfx950: the per-iteration
// sampling pass of m-Cubes.
//
// Work mapping: one lane per sub-cube at a time, persistent workgroups that
// stride through the g^d sub-cubes.  Because every random number is keyed by
// (seed; iteration, sub-cube, sample) rather than by thread, the mapping of
// sub-cubes to lanes does not change any sample point.
//
// Per sample (FP64, or FP32 for the map and the integrand in the FP32-eval
// path; no implicit contraction, fma only where written):
//   Philox4x32-10 blocks -> 52-bit uniforms -> stratified coordinate in bins
//   -> bin index, boundary and width from the LDS copy of the grid -> point
//   and Jacobian -> integrand -> I_k = f J / (m p) -> shifted per-cube sums
//   -> (V-Sample only) I_k^2 added to one LDS bin per axis.
// Per sub-cube: I_t and the unbiased variance estimate, accumulated per lane
// with error-free transformations.  Per workgroup: a fixed-order wave and
// workgroup reduction, then the totals go to this workgroup's slot of the
// partials array and the LDS histogram is added into one of the histogram
// accumulators, both merged after the pass (finalize or steps kernel).
#pragma once

#include <type_traits>

#include "fused.hpp"
#include "internal.hpp"

namespace mcubes {

// Read-only data reached through the constant address space: uniform loads
// become scalar loads, which the compiler may repeat instead of keeping every
// value in registers.  Only for memory that nothing writes while the kernel
// runs.
template <typename T>
using Const = __attribute__((address_space(4))) const T;


// The constants of axis j.  The single-integral kernel passes a volatile
// pointer: the compiler then reloads each constant where it is used instead of
// holding every axis's constants in scalar registers (which spilled them).
// With BATCH the pointer is instead made opaque once per axis, by an empty asm
// that the loads through it cannot move above: they still stay inside the
// loops, but they are no longer volatile, so the compiler merges the axis's
// loads and waits for them once rather than once per value (each wait also
// drains the LDS reads in flight).  That is 2-3% faster for the FP64
// Gaussian and table kernels and up to 2% slower for the others (more scalar
// spills), so those keep the per-use loads.
template <bool BATCH, typename CP>
__device__ __forceinline__ auto axis_consts(CP base, int j) {
    using P = std::remove_pointer_t<CP>;
    if constexpr (BATCH && std::is_volatile_v<P>) {
        auto p = const_cast<std::remove_volatile_t<P> *>(base + kConstStride * j);
        asm volatile("" : "+s"(p));
        return p;
    } else {
        return base + kConstStride * j;
    }
}

// ---------------------------------------------------------------- Philox4x32-10
// Salmon et al., SC'11: ten rounds of two 32x32->64 products, with the key
// advanced by the Weyl constants between rounds.  The key is uniform across
// the wavefront, so its schedule stays in scalar registers.  Each round's two
// three-way XORs are single v_bitop3_b32 instructions (truth table 0x96 is
// a ^ b ^ c).
//
// Of a block's counter (c, iteration, t_lo, t_hi) only t_lo differs between
// the lanes of a wavefront (see uniform_hi), and of the blocks of a sub-cube
// only c, so the first rounds split into what the sub-cube's blocks share
// (PhiloxCube, once per sub-cube) and what is uniform (scalar instructions):
// a block is left with the two XORs of round 2, two products and two XORs in
// round 3, and two of each in rounds 4 to 10, 16 products instead of 20.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kWeyl0 = 0x9E3779B9u, kWeyl1 = 0xBB67AE85u;

// The upper half of the sub-cube index, uniform across the wavefront: the
// lanes of a wave hold consecutive indices that start at a multiple of their
// number, so they never straddle a multiple of 2^32.
__device__ __forceinline__ uint32_t uniform_hi(uint64_t t) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(t >> 32));
}

// What every block of sub-cube t shares: the low word of round 1's second
// product, and both words of round 2's first.
struct PhiloxCube {
    uint32_t b1, h2, l2;
};

__device__ __forceinline__ PhiloxCube philox_cube(uint32_t tlo, uint32_t iter, uint32_t k0) {
    const uint64_t pb = (uint64_t)kPhiloxM1 * (uint64_t)tlo;
    const uint64_t pa = (uint64_t)kPhiloxM0 * (uint64_t)((uint32_t)(pb >> 32) ^ (iter ^ k0));
    return PhiloxCube{(uint32_t)pb, (uint32_t)(pa >> 32), (uint32_t)pa};
}

// Block c of a sub-cube: w[0..3].  c and thi are uniform.
__device__ __forceinline__ void philox_block(const PhiloxCube &q, uint32_t c, uint32_t thi, uint32_t k0,
                                             uint32_t k1, uint32_t *w) {
    // round 1 and round 2's second product: scalar
    const uint64_t pa1 = (uint64_t)kPhiloxM0 * (uint64_t)c;
    const uint64_t pb2 = (uint64_t)kPhiloxM1 * (uint64_t)((uint32_t)(pa1 >> 32) ^ thi ^ k1);
    k0 += kWeyl0;
    k1 += kWeyl1;
    uint32_t x0 = q.b1 ^ ((uint32_t)(pb2 >> 32) ^ k0);
    uint32_t x2 = q.h2 ^ ((uint32_t)pa1 ^ k1);
    k0 += kWeyl0;
    k1 += kWeyl1;
    // round 3
    uint64_t pa = (uint64_t)kPhiloxM0 * (uint64_t)x0;
    uint64_t pb = (uint64_t)kPhiloxM1 * (uint64_t)x2;
    x0 = (uint32_t)(pb >> 32) ^ ((uint32_t)pb2 ^ k0);
    x2 = xor3((uint32_t)(pa >> 32), q.l2, k1);
    uint32_t x1 = (uint32_t)pb, x3 = (uint32_t)pa;
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        k0 += kWeyl0;
        k1 += kWeyl1;
        pa = (uint64_t)kPhiloxM0 * (uint64_t)x0;
        pb = (uint64_t)kPhiloxM1 * (uint64_t)x2;
        x0 = xor3((uint32_t)(pb >> 32), x1, k0);
        x2 = xor3((uint32_t)(pa >> 32), x3, k1);
        x1 = (uint32_t)pb;
        x3 = (uint32_t)pa;
    }
    w[0] = x0;
    w[1] = x1;
    w[2] = x2;
    w[3] = x3;
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ float uniform(float x) { return __uint_as_float(uniform(__float_as_uint(x))); }
__device__ __forceinline__ double uniform(double x) {
    return __hiloint2double((int)uniform((uint32_t)__double2hiint(x)), (int)uniform((uint32_t)__double2loint(x)));
}

// (2X+1) 2^-53 for the 52-bit X = (whi << 20) | (wlo >> 12): the double with
// exponent 0 and mantissa X is 1 + X 2^-52; subtracting 1 - 2^-53 is exact
// (Sterbenz), so the result is exactly the open-interval uniform.
__device__ __forceinline__ double uniform53(uint32_t whi, uint32_t wlo) {
    // both words are funnel shifts of a 64-bit pair: {0x3FF, whi} >> 12 is
    // 0x3FF00000 | (whi >> 12), and {whi, wlo} >> 12 is (whi << 20) | (wlo >> 12)
    const uint32_t hi = __builtin_amdgcn_alignbit(0x3FFu, whi, 12);
    const uint32_t lo = __builtin_amdgcn_alignbit(whi, wlo, 12);
    return __hiloint2double((int)hi, (int)lo) - 0x1.fffffffffffffp-1;
}

// ---------------------------------------------------------------- FP32-eval helpers

// (2 (w >> 9) + 1) 2^-24: the float with exponent 0 and mantissa w >> 9 is
// 1 + (w >> 9) 2^-23; subtracting 1 - 2^-24 is exact (Sterbenz).
__device__ __forceinline__ float uniform24(uint32_t w) {
    // {0x7F, w} >> 9 is 0x3F800000 | (w >> 9)
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, w, 9)) - 0x1.fffffep-1f;
}

// Arithmetic of the evaluation precision R (double for the FP64 path, float
// for FP32 evaluation): each is a single correctly rounded IEEE operation.
__device__ __forceinline__ double rfma(double a, double b, double c) { return __fma_rn(a, b, c); }
__device__ __forceinline__ float rfma(float a, float b, float c) { return __fmaf_rn(a, b, c); }
__device__ __forceinline__ double rfloor(double a) { return floor(a); }
__device__ __forceinline__ float rfloor(float a) { return floorf(a); }
__device__ __forceinline__ double rmin(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float rmin(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double rmax(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float rmax(float a, float b) { return fmaxf(a, b); }

// fma(q, r, C) with the constant C (given by its bits) written into a scalar
// register pair right where it is used: the two moves are asm that cannot leave
// the loops, and the product is the three-operand instruction, so C is
// held neither in vector registers for the whole kernel (and copied from there
// into the accumulator of a two-operand fma) nor in scalar ones (which spill).
template <uint64_t C>
__device__ __forceinline__ double fma_const(double q, double r) {
    uint32_t lo, hi;
    asm volatile("s_mov_b32 %0, %1" : "=s"(lo) : "i"((int32_t)(uint32_t)C));
    asm volatile("s_mov_b32 %0, %1" : "=s"(hi) : "i"((int32_t)(uint32_t)(C >> 32)));
    const double c = __hiloint2double((int)hi, (int)lo);
    double out;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(out) : "v"(q), "v"(r), "s"(c));
    return out;
}

// e^-a for a >= 0 (or NaN): a = -n ln 2 - r with |r| <= ln 2 / 2, then
// 1 + r + r^2/2 + r^3 q(r) by Horner's rule, scaled by 2^n; 0 beyond 1075, where
// e^-a rounds to 0.  q is the polynomial of degree nine with the smallest
// largest relative error of the sum there (Remez exchange, 7.5e-20), so only the
// roundings count: in ulps of a normal result at most 0.5 of the last step,
// 0.18 of the sum it multiplies by r, 0.20 of r and 0.04 of the rest, 0.90 in all
// where they meet.  Over 1e8 draws at most 0.873, root mean square 0.3013; the device
// library's exp 0.886 and 0.3017 (degree eight, one step less: 1.046 and 0.3047).  That exp,
// no longer, kept its coefficients in vector registers and copied each into the
// accumulator of a two-operand fma.
__device__ __forceinline__ double exp_neg(double a) {
    const double n = rint(a * -0x1.71547652b82fep+0);
    double r = __fma_rn(n, -0x1.62e42fefa39efp-1, -a);  // exact
    r = __fma_rn(n, -0x1.abc9e3b39803fp-56, r);
    double q = fma_const<0x3e5af7a29407b03dull>(0x1.20d15d9f70984p-29, r);
    q = fma_const<0x3e927e40c0273beaull>(q, r);
    q = fma_const<0x3ec71dde7ba27f8eull>(q, r);
    q = fma_const<0x3efa01a01fc75a44ull>(q, r);
    q = fma_const<0x3f2a01a01b6f1334ull>(q, r);
    q = fma_const<0x3f56c16c16c07ee5ull>(q, r);
    q = fma_const<0x3f8111111110e33full>(q, r);
    q = fma_const<0x3fa555555555556full>(q, r);
    q = fma_const<0x3fc555555555555dull>(q, r);
    q = __fma_rn(q, r, 0.5);
    q = __fma_rn(q, r, 1.0);
    q = __fma_rn(q, r, 1.0);
    const double e = ldexp(q, (int)n);
    return a > 1075.0 ? 0.0 : e;
}
__device__ __forceinline__ float exp_neg(float a) { return expf(-a); }

// The bin of the stratified coordinate z >= 0 (in bins) and the fraction inside
// it, the bin clamped to the last one and the fraction to 1 there: once
// z >= nb, z - (nb-1) is at least 1 and the clamp makes it exactly 1; otherwise
// z - floor(z) < 1 is exact.  The clamp to [0, 1] is the output modifier of
// the subtraction, free.  FP64 truncates to the integer first and converts
// back (floor and a FP64 minimum would cost 2 cycles more than the integer
// minimum and the conversion); in FP32 floor and minimum are the cheaper half.
__device__ __forceinline__ double bin_of(double z, int last, double, int &i) {
    i = min((int)z, last);
    return fmin(fmax(z - (double)i, 0.0), 1.0);
}
__device__ __forceinline__ float bin_of(float z, int, float lastf, int &i) {
    const float fz = rmin(rfloor(z), lastf);
    i = (int)fz;
    return fminf(fmaxf(z - fz, 0.0f), 1.0f);
}

// The same in FP64 for untraced passes: z clamped to zlast, the last double below
// nb, first, after which one instruction (v_fract_f64) is z - floor(z), without the
// conversion back.  The fraction differs from bin_of's only where z rounded up to
// nb: 1 - 2^-44 (nb = 500) rather than 1, each within the rounding of z of the true
// one, which lies below 1 (at 12 intervals one axis value in 2^53 or so).  With the Jacobian's one product per axis
// (J0 in cube_pass), 12 instead of 18 issue cycles per sample and axis: d = 8
// corner peak, 1e9 samples 7715 -> 7450 us; d = 9 Gaussian, 3e7, No-Adjust 271 -> 266;
// a mixed batch of 192 (bin_below only) 9.81 -> 9.62 ms.  Passes that spread a
// sub-cube over lanes (kSplit, kFused) are bound by latency and keep the above:
// d = 10 tables, 1e6 samples 35.1 us against 35.5.
__device__ __forceinline__ double bin_below(double z, double zlast, int &i) {
    const double zb = __builtin_fmin(z, zlast);
    i = (int)zb;
    return __builtin_amdgcn_fract(zb);
}

// ---------------------------------------------------------------- integrands

template <typename R>
__device__ __forceinline__ R lerp(R a, R b, R t) {
    return rfma(t, b - a, a);
}

// Bilinear interpolation in one 256x256 table, node (a,b) at (a/255, b/255),
// the edge cell extended outside the unit square, in two parts: table_cell
// finds the cell of (x, y) and loads its four nodes, interpolate combines
// them.  The integrand fetches each table's cell as soon as its two
// coordinates are known, so the loads are in flight while the remaining axes
// and the exponential are computed; the arithmetic is that of one bilinear
// interpolation, in the same order.
template <typename R>
struct TableCell {
    R t00, t01, t10, t11, tx, ty;
};

// Device layout of the two tables, one after the other.  FP64: row-major,
// node (a, b) at a * 256 + b; the two nodes of a cell's row are adjacent, so
// a cell is two 16-byte loads.  FP32-eval: row pairs, element 2 (a * 256 + b)
// holding node (a, b) and the next one node (a + 1, b) (0 for a = 255), so a
// cell's four nodes are four consecutive floats, one 16-byte load instead of
// two 8-byte ones (2% faster; the same layout in FP64 measured 0.5% slower).
template <typename R>
constexpr int kTableStride = std::is_same<R, float>::value ? 2 * kTableN * kTableN : kTableN * kTableN;

// The cell of a table coordinate u (in nodes) and the offset in it, the edge
// cell extended outside [0, 255].  FP64 truncates, clamps the integer and
// converts it back (truncation differs from floor only below 0, where the
// clamp makes both 0), one instruction less than floor and two FP64 clamps; in
// FP32 floor and the three-way median are the cheaper half.
__device__ __forceinline__ int table_axis(double u, double &t) {
    int a;  // the instruction itself: it saturates, where C++ leaves large u and NaN undefined
    asm("v_cvt_i32_f64 %0, %1" : "=v"(a) : "v"(u));
    a = min(max(a, 0), kTableN - 2);
    t = u - (double)a;
    return a;
}
__device__ __forceinline__ int table_axis(float u, float &t) {
    const float fa = rmin(rmax(rfloor(u), 0.0f), (float)(kTableN - 2));
    t = u - fa;
    return (int)fa;
}

template <typename R>
__device__ __forceinline__ TableCell<R> table_cell(const R *__restrict__ T, R x, R y) {
    TableCell<R> c;
    const int a = table_axis(x * R(kTableN - 1), c.tx);
    const int b = table_axis(y * R(kTableN - 1), c.ty);
    // a 32-bit byte offset from the uniform base: one scalar and one vector
    // address register, no 64-bit address arithmetic
    const uint32_t off = (uint32_t)(a * kTableN + b) * 8u;
    const char *base = reinterpret_cast<const char *>(T);
    if constexpr (std::is_same<R, float>::value) {
        // two 8-byte-aligned pairs, which the compiler merges into one load
        const float2 *q = reinterpret_cast<const float2 *>(base + off);
        const float2 lo = q[0], hi = q[1];
        c.t00 = lo.x;
        c.t10 = lo.y;
        c.t01 = hi.x;
        c.t11 = hi.y;
    } else {
        const double *q = reinterpret_cast<const double *>(base + off);
        c.t00 = q[0];
        c.t01 = q[1];
        c.t10 = q[kTableN];
        c.t11 = q[kTableN + 1];
    }
    return c;
}

template <typename R>
__device__ __forceinline__ R interpolate(const TableCell<R> &c) {
    return lerp(lerp(c.t00, c.t10, c.tx), lerp(c.t01, c.t11, c.tx), c.ty);
}

// The integrand, accumulated axis by axis in ascending order so that the
// point itself need not stay in registers:
//   Gaussian product  acc = sum_j t_j^2 by fma, t_j = (x_j - c_j) * (1/w_j); f = exp(-acc)
//   corner peak       S = 1 + sum_j a_j x_j by fma; f = 1 / S^(D+1), the power by
//                     left-to-right binary powering, one correctly rounded division
//   tables            the Gaussian product times T1(x_1, x_2) times T2(x_3, x_4)
// EARLY (tables only): fetch each table's cell as soon as its coordinates are
// known rather than at the end; the loads then overlap the remaining axes and
// the exponential, at the price of registers for the eight nodes.  Kernels
// that inline many cases into one register allocation leave it off.
template <int F, int D, typename R, bool EARLY>
struct Integrand {
    R acc;
    R x0, x1, x2, x3;        // table coordinates (tables only)
    TableCell<R> c1, c2;     // the two tables' cells (tables, EARLY only)
    const R *T;              // the two tables, one after the other (tables only)

    __device__ __forceinline__ explicit Integrand(const void *tables)
        : acc(F == 2 ? R(1) : R(0)), x0(0), x1(0), x2(0), x3(0), c1(), c2(),
          T(static_cast<const R *>(tables)) {}

    template <typename CP>
    __device__ __forceinline__ void axis(int j, R xj, CP cj) {
        if constexpr (F == 1 || F == 3) {
            const R t = (xj - cj[3]) * cj[4];
            acc = rfma(t, t, acc);
        } else if constexpr (F == 2) {
            acc = rfma(cj[3], xj, acc);
        }
        if constexpr (F == 3) {
            if (j == 0) x0 = xj;
            if (j == 1) x1 = xj;
            if (j == 2) x2 = xj;
            if (j == 3) x3 = xj;
            if constexpr (EARLY) {
                if (j == 1) c1 = table_cell(T, x0, x1);
                if (j == 3) c2 = table_cell(T + kTableStride<R>, x2, x3);
            }
        }
    }

    template <typename A>
    __device__ __forceinline__ R value(const A &a) const {
        if constexpr (F == 0) {
            return R(a.cval);
        } else if constexpr (F == 1) {
            return exp_neg(acc);
        } else if constexpr (F == 2) {
            constexpr unsigned e = (unsigned)(D + 1);
            constexpr int top = 31 - __builtin_clz(e);
            R pw = acc;
#pragma unroll
            for (int bit = top - 1; bit >= 0; --bit) {
                pw = pw * pw;
                if ((e >> bit) & 1u) pw = pw * acc;
            }
            return R(1) / pw;
        } else {
            static_assert(D >= 4, "table integrand needs four axes");
            const R G = exp_neg(acc);
            const R T1 = interpolate(EARLY ? c1 : table_cell(T, x0, x1));
            const R T2 = interpolate(EARLY ? c2 : table_cell(T + kTableStride<R>, x2, x3));
            return (G * T1) * T2;
        }
    }
};

// ---------------------------------------------------------------- compensated sums

// s + c += v with the exact rounding error of s + v kept in c (Knuth's TwoSum).
__device__ __forceinline__ void two_sum_add(double &s, double &c, double v) {
    const double t = s + v;
    const double bp = t - s;
    const double e = (s - (t - bp)) + (v - bp);
    s = t;
    c += e;
}

__device__ __forceinline__ void two_sum_merge(double &s, double &c, double s2, double c2) {
    const double t = s + s2;
    const double bp = t - s;
    const double e = (s - (t - bp)) + (s2 - bp);
    s = t;
    c = (c + c2) + e;
}

// ---------------------------------------------------------------- LDS layout

// Per workgroup: the grid, then (V-Sample only) the d x nb histogram.  FP64
// keeps each axis's nb+1 boundaries; FP32 keeps per bin its left boundary and
// width, each rounded once from FP64.  (The per-axis constants are read with
// scalar loads from device memory; see Const.)
template <bool F32>
__host__ __device__ constexpr size_t lds_grid_bytes(int d, int nb) {
    return F32 ? (size_t)d * nb * 2 * sizeof(float) : (size_t)d * (nb + 1) * sizeof(double);
}

// ---------------------------------------------------------------- building blocks

template <bool F32>
using real_t = typename std::conditional<F32, float, double>::type;

// The workgroup's LDS regions for an integral of dimension d with nb bins.
template <bool F32>
struct LdsView {
    real_t<F32> *grid;
    double *hist;
    __device__ LdsView(double *lds, int d, int nb) {
        char *base = reinterpret_cast<char *>(lds);
        grid = reinterpret_cast<real_t<F32> *>(base);
        hist = reinterpret_cast<double *>(base + lds_grid_bytes<F32>(d, nb));
    }
};

// LDS addresses.  A sample's bin on axis j is one 8-byte grid entry (FP64: the
// left boundary, followed by the right one; FP32: the float pair), whose LDS
// address also leads to the bin's histogram entry: row j of the grid starts j
// entries further into its region in FP64 (rows of nb + 1) than row j of the
// histogram, and not at all in FP32 (rows of nb), so the histogram entry lies
// at a distance from the grid entry that is the same for every bin and axis up
// to an instruction offset of 8 (D - 1 - j) bytes (to_hist).  One two-cycle
// addition per contribution replaces a four-cycle shift-and-add.
using LdsDouble = __attribute__((address_space(3))) double;
using LdsWord = __attribute__((address_space(3))) uint64_t;

__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)(const char *)p;
}

// The LDS address of entry i of a grid row that starts at row_address; opaque,
// so that the address is kept rather than formed again for the histogram.
__device__ __forceinline__ uint32_t cell_address(uint32_t row_address, int i) {
    uint32_t a = row_address + ((uint32_t)i << 3);
    asm("" : "+v"(a));
    return a;
}

// A grid entry as it lies in LDS: the left boundary and the right one (FP64)
// or the width (FP32); read_cell gives the width in both.
__device__ __forceinline__ void load_cell(uint32_t cell, double &left, double &right) {
    LdsDouble *B = (LdsDouble *)cell;
    left = __hip_atomic_load(B, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    right = __hip_atomic_load(B + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void load_cell(uint32_t cell, float &left, float &width) {
    const uint64_t B = *(const LdsWord *)cell;  // one 8-byte read
    left = __uint_as_float((uint32_t)B);
    width = __uint_as_float((uint32_t)(B >> 32));
}
template <typename R>
__device__ __forceinline__ void read_cell(uint32_t cell, R &left, R &width) {
    load_cell(cell, left, width);
    if constexpr (!std::is_same<R, float>::value) width = width - left;
}

// (COPIES: cell is the bin's entry in row 0, to_hist the row's distance.)
template <int D, bool F32, bool COPIES>
__device__ __forceinline__ void add_bin(uint32_t cell, uint32_t to_hist, int j, double v) {
    LdsDouble *h = (LdsDouble *)(cell + to_hist) + (F32 || COPIES ? 0 : D - 1 - j);
    __hip_atomic_fetch_add(h, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Copies the integral's grid into LDS and clears the histogram.  Callers
// synchronise the workgroup afterwards.  (A is SampleArgs, possibly in the
// constant address space: see the batched kernel.)
template <int D, bool F32, typename A>
__device__ __forceinline__ void load_lds(const A &a, const LdsView<F32> &v) {
    const int nb = a.nb, row = nb + 1, tid = threadIdx.x, nthr = blockDim.x;
    if constexpr (F32) {
        for (int i = tid; i < D * nb; i += nthr) {
            const int j = i / nb, b = i - j * nb;
            const double *B = a.grid + j * row + b;
            v.grid[2 * i] = (float)B[0];
            v.grid[2 * i + 1] = (float)(B[1] - B[0]);
        }
    } else {
        for (int i = tid; i < D * row; i += nthr) v.grid[i] = a.grid[i];
    }
    if (a.hist)
        for (int i = tid; i < D * nb * a.hist_copies; i += nthr) v.hist[i] = 0.0;
}

// Whether the one-sample path computes every axis's bin and issues every
// grid read before the rest of the sample (GF in cube_pass).  Each axis's
// constants are scalar loads whose wait also waits for the LDS reads in
// flight, so axis by axis every grid read was waited for on its own; in two
// phases they overlap.  Taken for the FP64 Gaussian and table kernels where
// the values held across the phases keep the occupancy and add no spill:
// 3-4% faster at d = 4, 2-3% at d = 6 to 8 (the d = 6 table kernel 1.024 ->
// 0.993 ms), 1% for the tables at d = 7, and for the FP32-eval table kernel
// at d = 6 together with the priority hint of cube_pass held until the
// integrand value (1.5%; 3% slower without the hint); the corner-peak
// kernels lose occupancy (d = 8: 9% slower; 4% with the hint), and d >= 10
// would spill.
template <int F, int D, bool F32>
constexpr bool kGridFirst =
    (!F32 && ((F == 1 && (D == 3 || D == 4 || (D >= 6 && D <= 9))) || (F == 3 && D >= 4 && D <= 7))) ||
    (F32 && F == 3 && D == 6);

// Whether cube_pass evaluates the samples of a sub-cube two at a time.  Two
// independent evaluations interleave and hide each other's LDS and
// transcendental latency, but both must fit in registers: in FP32 evaluation
// they do (up to d = 11, d = 8 with tables); in FP64 the pair spills to
// scratch memory (over 1 GB of HBM writes per launch at d = 6), so FP64
// keeps one sample at a time.  The FP32 table kernel at d = 6 also keeps one:
// the pair needs 86 VGPRs, which allows one 1024-thread workgroup per CU (4
// waves per SIMD), one sample at a time 69, which allows two 768-thread
// workgroups (6 waves per SIMD, the LDS limit) and is 11% faster; the pair
// had been 6% faster at the 4-wave shape.
template <int F, int D, bool F32>
constexpr bool kPairSamples = F32 && (F == 3 ? D <= 8 && D != 6 : D <= 11);

// Whether the single-integral kernel keeps each axis's lower bound in vector
// registers for the whole launch.  The point x = lo + span xu is one fma with
// two scalar operands otherwise, which the hardware cannot read in one
// instruction, so every sample moved lo into a vector register first (two
// moves per axis in FP64, one in FP32).  Taken for the FP64 Gaussian and
// table kernels of d = 6..8 (5% fewer VALU instructions at d = 6 and 8,
// 1.5-1.7% faster) and the FP32 table kernel at d = 6 (1.4% faster), which
// keep their waves per SIMD; at lower d the extra registers cost waves, at
// higher d they spill, and the d = 8 corner-peak and FP32 d = 8 kernels
// would lose the two workgroups per CU they run at.
template <int F, int D, bool F32>
constexpr bool kLowInVgpr = F32 ? (F == 3 && D == 6) : ((F == 1 || F == 3) && D >= 6 && D <= 8);

// The waves per SIMD the compiler is told a kernel runs at, where that is
// fixed by its launch (amdgpu_waves_per_eu(w, w)), so that it schedules for
// that occupancy rather than for a higher one the kernel cannot reach; 0: the
// compiler's own range (1 to 8 waves, which compiles to the same code as no
// attribute).  4 for the FP64 Gaussian kernels of d = 6..8 and table kernels
// of d = 6, 7 (108-128 VGPRs, one 1024-thread workgroup per CU either way):
// 0.6% faster at d = 6 with the tables, 0.8% at d = 8 with the Gaussian (at
// d = 8 with the tables it would spill 12 bytes).  6 for the FP32 table
// kernel at d = 6 (two 72 KB workgroups of 768 threads per CU): 0.6% faster;
// the d = 8 corner-peak kernels, also at 6 by their LDS, measured 0.5-1.5%
// slower with it.
template <int F, int D, int KIND, bool F32>
constexpr int kFixedWaves =
    KIND != kPlain && KIND != kPerAxis && KIND != kCopies ? 0
          : (!F32 && ((F == 1 && D >= 6 && D <= 8) || (F == 3 && (D == 6 || D == 7)))) ? 4
          : (F32 && F == 3 && D == 6) ? 6
                                      : 0;

// The slow axes of a staged launch (the NS last): all sub-cubes that the
// workgroup has in hand share their digits, so those are scalars, the grid in
// LDS is the window of bins their stratum can reach, and the histogram that
// window with 2^stage_shift copies of every bin side by side, lane by lane (32,
// one per lane of a half-wave, where the LDS holds them).
template <typename R, int NS>
struct SlowAxes {
    R c[NS ? NS : 1];              // the digits
    uint32_t row[NS ? NS : 1];     // LDS address that grid entry 0 would have
    uint32_t stage[NS ? NS : 1];   // this lane's copy of histogram entry 0, likewise
};

// All p samples of sub-cube t (digits dig): returns I_t and var_t, adds the bin
// contributions to the LDS histogram when collecting them, and records the
// cube in the trace when tracing.  PAIR: evaluate the samples two at a time
// (kPairSamples for a kernel of its own; kernels that inline many cases into
// one register allocation leave it off).  EARLY: see Integrand.  LOV: lov
// holds the axes' lower bounds in vector registers (kLowInVgpr); otherwise
// they are read with the other constants.  (A compile-time choice: a null
// pointer tested at run time, though folded away, changed the FP32 d = 8
// kernels' register allocation from 72 to 90.)  GF: see kGridFirst.  PRIO:
// the one-sample path raises the wave's priority for the first part of each
// sample (the pair path always does).
template <int F, int D, bool TRACE, bool F32, bool PAIR, bool EARLY, bool LOV = false, bool GF = false,
          bool PRIO = false, bool COPIES = false, bool SPLIT = false, int NS = 0, bool UNIT = false, bool J0 = false,
          typename A, typename CP>
__device__ __forceinline__ void cube_pass(const A &a, const LdsView<F32> &v, CP sC, uint64_t t,
                                          const uint32_t (&dig)[D - NS], double &It, double &vt,
                                          bool &bad, const real_t<F32> *lov = nullptr,
                                          const SlowAxes<real_t<F32>, NS> &slow = {}) {
    using R = real_t<F32>;
    constexpr int K = D - NS;  // axes below K are each lane's own
    constexpr bool kBatchConsts = !F32 && (F == 1 || F == 3);  // see axis_consts
    constexpr int NBLK = (D + 1) / 2;                      // blocks in the counter layout
    constexpr int NUSED = F32 ? (D + 3) / 4 : NBLK;        // blocks this precision needs
    const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
    const int nb = a.nb, row = F32 ? nb : nb + 1, rec = 3 * D + 2;
    const R s = R(F32 ? a.s32 : a.s);
    const int last = nb - 1;
    const R lastr = R(last);
    const uint32_t grid0 = lds_address(v.grid), row_bytes = (uint32_t)row * 8u;
    // from a grid entry to its bin's histogram entry (see above); with two
    // histogram copies the upper half of each wave adds into the second, so at
    // most half as many lanes add into one bin at once
    uint32_t to_hist = lds_address(v.hist) - grid0 - (F32 ? 0u : 8u * (D - 1));
    if (!COPIES && a.hist_copies > 1 && (threadIdx.x & 32)) to_hist += (uint32_t)((D - NS) * nb) * 8u;
    // COPIES: the copies of a bin lie next to each other (row, bin, copy), and a
    // lane adds into copy lane mod copies
    const uint32_t copy_sh = COPIES ? 3u + (uint32_t)a.copy_shift : 3u;
    const uint32_t lane_hist =
        COPIES ? lds_address(v.hist) + ((threadIdx.x & ((1u << a.copy_shift) - 1u)) << 3) : 0u;
    const uint32_t hist_row = (uint32_t)nb << copy_sh;
    // SPLIT: lane q of a group of 2^lsplit neighbours takes the samples q, q +
    // 2^lsplit, ... of the group's sub-cube
    const int kstep = SPLIT ? 1 << a.lsplit : 1;
    const int kfirst = SPLIT ? (int)(threadIdx.x & (uint32_t)(kstep - 1)) : 0;

    R cd[D];
#pragma unroll
    for (int j = 0; j < D; ++j) cd[j] = j < K ? R(dig[j]) : slow.c[j < K ? 0 : j - K];
    // the largest double below nb
    const double zlast = uniform(__longlong_as_double(__double_as_longlong((double)nb) - 1));
    // the bin of axis j and the fraction inside it
    auto bin_at = [&](int j, const uint32_t *w, R &u, int &i) -> R {
        if constexpr (F32) u = uniform24(w[j]);
        else u = uniform53(w[j], w[D + j]);
        const R z = (cd[j] + u) * s;
        if constexpr (F32 || TRACE || SPLIT) return bin_of(z, last, lastr, i);
        else return bin_below(z, zlast, i);
    };
    const R first_J = J0 ? R(a.j0) : R(1);
    // the Jacobian: with J0 the volume and the bins are its first factor
    auto times_width = [&](R J, R width, const auto &cj) -> R {
        if constexpr (J0) return J * width;
        else return J * (width * (UNIT ? R(nb) : cj[2]));
    };
    const uint32_t stage_sh = 3u + (uint32_t)a.stage_shift;
    auto row_address = [&](int j) { return j < K ? grid0 + j * row_bytes : slow.row[j < K ? 0 : j - K]; };
    // what add_bin takes for bin i of axis j, whose grid cell is at `cell`
    auto target_of = [&](int j, int i, uint32_t cell) -> uint32_t {
        if (COPIES) return ((uint32_t)i << copy_sh) + lane_hist;
        return j < K ? cell : slow.stage[j < K ? 0 : j - K] + ((uint32_t)i << stage_sh);
    };
    auto add_to = [&](uint32_t target, int j, double sq) {
        if (j >= K) add_bin<D, F32, true>(target, 0u, j, sq);
        else add_bin<D, F32, COPIES>(target, COPIES ? j * hist_row : to_hist, j, sq);
    };
    const uint32_t thi = NS ? 0u : uniform_hi(t);  // (staged launches: below 2^32)
    const PhiloxCube pc = philox_cube((uint32_t)t, a.iter, k0);
    const bool traced = TRACE && (int64_t)t >= a.t0 && (int64_t)t < a.t1;

    double I0 = 0.0, S1 = 0.0, S2 = 0.0;
    if constexpr (PAIR) {
        // One sample: its value I_k and, per axis, the grid cell or histogram
        // entry that add_bin takes (and its trace record).
        auto point = [&](int k, uint32_t (&target)[D]) -> double {
            // raised wave priority while the sample's random words, bins and
            // grid reads are formed, back to normal before its integrand
            // value (see the one-sample path below; FP32-eval Gaussian and
            // corner-peak kernels 2-3% faster)
            __builtin_amdgcn_s_setprio(1);
            uint32_t w[4 * NUSED];
#pragma unroll
            for (int b = 0; b < NUSED; ++b)
                philox_block(pc, (uint32_t)(k * NBLK + b), thi, k0, k1, w + 4 * b);
            Integrand<F, D, R, EARLY> fx(a.tables);
            R J = first_J;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                R u;
                int i;
                const R frac = bin_at(j, w, u, i);
                const uint32_t cell = cell_address(row_address(j), i);
                target[j] = target_of(j, i, cell);
                R left, width;
                read_cell(cell, left, width);
                const R xu = rfma(frac, width, left);
                const auto cj = axis_consts<kBatchConsts>(sC, j);
                R xj;
                if constexpr (UNIT)
                    xj = xu;  // lo = 0, span = 1: the product and the sum are exact
                else if constexpr (LOV)
                    xj = rfma(cj[1], xu, lov[j]);
                else
                    xj = rfma(cj[1], xu, cj[0]);
                J = times_width(J, width, cj);
                fx.axis(j, xj, cj);
                if (traced) {
                    double *r = a.trace + ((t - a.t0) * (uint64_t)a.p + k) * rec;
                    r[j] = (double)u;
                    r[D + j] = (double)i;
                    r[2 * D + j] = (double)xj;
                }
            }
            __builtin_amdgcn_s_setprio(0);
            const R f = fx.value(a);
            if (traced) {
                double *r = a.trace + ((t - a.t0) * (uint64_t)a.p + k) * rec;
                r[3 * D] = (double)J;
                r[3 * D + 1] = (double)f;
            }
            // f J, not f alone: in FP32 evaluation the Jacobian can overflow
            const double Fv = (double)f * (double)J;
            bad |= !isfinite(Fv);
            return Fv * a.inv;
        };
        // shifted sums in sample order
        // (for k == 0 the deviation is exactly +0 and leaves S1 = S2 = +0)
        auto accumulate = [&](int k, double Ik) {
            if (k == kfirst) I0 = Ik;
            const double dev = Ik - I0;
            S1 = S1 + dev;
            S2 = __fma_rn(dev, dev, S2);
        };
        auto add_bins = [&](const uint32_t (&cell)[D], double Ik) {
            if (a.hist) {
                const double sq = Ik * Ik;
                const int axes = a.one_d ? 1 : D;
#pragma unroll
                for (int j = 0; j < D; ++j)
                    if (j < axes) add_to(cell[j], j, sq);
            }
        };
        {
            // both points (grid reads included) before either sample's histogram
            // atomics, so that the two evaluations can interleave
            int k = kfirst;
            for (; k + kstep < a.p; k += 2 * kstep) {
                uint32_t cell0[D], cell1[D];
                const double Ia = point(k, cell0);
                const double Ib = point(k + kstep, cell1);
                accumulate(k, Ia);
                accumulate(k + kstep, Ib);
                add_bins(cell0, Ia);
                add_bins(cell1, Ib);
            }
            if (k < a.p) {
                uint32_t cell0[D];
                const double Ia = point(k, cell0);
                accumulate(k, Ia);
                add_bins(cell0, Ia);
            }
        }
    } else {
        // the same steps one sample at a time, written out in the loop: the
        // batched kernel, which inlines every case, allocates fewer registers
        // for this form than for the lambda one
        for (int k = kfirst; k < a.p; k += kstep) {
            // PRIO: the wave runs at raised priority from the start of a
            // sample until its integrand value.  s_setprio only orders issue
            // among the waves of a SIMD; favouring the waves that are still on
            // their way to their grid reads and table loads puts more of them
            // in flight while the others compute.  Taken with the two phases
            // (FP64 table and Gaussian kernels 2-5% faster), where phase 1
            // runs a level higher still (another 0.3-1.2%), and in the
            // batched kernel (FP32-eval 1%); the one-phase single-integral
            // kernels of this path, FP64 corner peak and FP32-eval tables at
            // d = 6, gained nothing or lost up to 2%.
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(GF ? 2 : 1);
            uint32_t w[4 * NUSED];
#pragma unroll
            for (int b = 0; b < NUSED; ++b)
                philox_block(pc, (uint32_t)(k * NBLK + b), thi, k0, k1, w + 4 * b);
            Integrand<F, D, R, EARLY> fx(a.tables);
            uint32_t cell[D];  // grid cells, or (COPIES) histogram entries
            R J = first_J;
            // GF: every axis's bin and grid read first, then the rest axis by
            // axis, so that the grid reads are in flight together rather
            // than each waited for before the next is issued (see kGridFirst)
            R gf_frac[GF ? D : 1], gf_left[GF ? D : 1], gf_right[GF ? D : 1];
            if constexpr (GF) {
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    R uj;
                    int i;
                    gf_frac[j] = bin_at(j, w, uj, i);
                    cell[j] = cell_address(row_address(j), i);
                    load_cell(cell[j], gf_left[j], gf_right[j]);
                    cell[j] = target_of(j, i, cell[j]);
                }
                __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of their uses
                if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
            }
#pragma unroll
            for (int j = 0; j < D; ++j) {
                R u = R(0), frac, left, width;
                if constexpr (GF) {
                    if (traced) {
                        if constexpr (F32) u = uniform24(w[j]);
                        else u = uniform53(w[j], w[D + j]);
                    }
                    frac = gf_frac[j];
                    left = gf_left[j];
                    if constexpr (F32) width = gf_right[j];
                    else width = gf_right[j] - left;
                } else {
                    int i;
                    frac = bin_at(j, w, u, i);
                    cell[j] = cell_address(row_address(j), i);
                    read_cell(cell[j], left, width);
                    cell[j] = target_of(j, i, cell[j]);
                }
                const R xu = rfma(frac, width, left);
                const auto cj = axis_consts<kBatchConsts>(sC, j);
                R xj;
                if constexpr (UNIT)
                    xj = xu;  // lo = 0, span = 1: the product and the sum are exact
                else if constexpr (LOV)
                    xj = rfma(cj[1], xu, lov[j]);
                else
                    xj = rfma(cj[1], xu, cj[0]);
                J = times_width(J, width, cj);
                fx.axis(j, xj, cj);
                if (traced) {
                    double *r = a.trace + ((t - a.t0) * (uint64_t)a.p + k) * rec;
                    r[j] = (double)u;
                    r[D + j] = (double)((cell[j] - (grid0 + j * row_bytes)) >> 3);
                    r[2 * D + j] = (double)xj;
                }
            }
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
            const R f = fx.value(a);
            const double Fv = (double)f * (double)J;
            bad |= !isfinite(Fv);
            const double Ik = Fv * a.inv;
            if (k == kfirst) I0 = Ik;
            {
                const double dev = Ik - I0;  // exactly +0 for the first: S1, S2 stay +0
                S1 = S1 + dev;
                S2 = __fma_rn(dev, dev, S2);
            }
            if (a.hist) {
                const double sq = Ik * Ik;
                const int axes = a.one_d ? 1 : D;
#pragma unroll
                for (int j = 0; j < D; ++j)
                    if (j < axes) add_to(cell[j], j, sq);
            }
            if (traced) {
                double *r = a.trace + ((t - a.t0) * (uint64_t)a.p + k) * rec;
                r[3 * D] = (double)J;
                r[3 * D + 1] = (double)f;
            }
        }
    }
    if constexpr (SPLIT) {
        if (kstep > 1) {
            // the group's sums: each lane's, shifted from its own first value to
            // the sub-cube's (that of the group's first lane), then a butterfly
            const int lane = threadIdx.x & 63;
            const double c0 = __shfl(I0, lane & ~(kstep - 1), 64);
            const double n = (double)((a.p - kfirst + kstep - 1) >> a.lsplit);
            const double dd = I0 - c0;
            S2 = __fma_rn(n * dd, dd, __fma_rn(2.0 * dd, S1, S2));
            S1 = __fma_rn(n, dd, S1);
            for (int off = kstep >> 1; off >= 1; off >>= 1) {
                S1 = S1 + __shfl_xor(S1, off, 64);
                S2 = S2 + __shfl_xor(S2, off, 64);
            }
            I0 = c0;
        }
    }
    It = __fma_rn(a.pd, I0, S1);
    const double num = __fma_rn(-S1, S1, a.pd * S2);
    vt = num * a.inv_pm1;
    if (vt < 0.0) vt = 0.0;
    if (SPLIT && kfirst != 0) It = vt = 0.0;  // the group's first lane counts the sub-cube
    if (traced) {
        double *r = a.trace + (uint64_t)(a.t1 - a.t0) * (uint64_t)a.p * rec + (t - a.t0) * 2;
        r[0] = It;
        r[1] = vt;
    }
}

// dig += step digit by digit in base g (the carry out of the top digit is
// dropped: the caller's cube index tells whether the lane is done).
template <int D>
__device__ __forceinline__ void odometer_add(uint32_t (&dig)[D], const int32_t *step, uint32_t g) {
    uint32_t carry = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const uint32_t v = dig[j] + (uint32_t)step[j] + carry;  // < 2g + 1 <= 2^31 + 1
        carry = v >= g ? 1u : 0u;
        dig[j] = carry ? v - g : v;
    }
}

// The digits of t in base g.  Below 2^32 each division is a product with
// gmagic = ceil(2^64 / g), whose upper word is the exact quotient for 32-bit t
// (two multiply-adds, where a 64-bit division takes about a hundred
// instructions: for ten digits that was longer than sampling a sub-cube).
template <int D>
__device__ __forceinline__ void digits_of32(uint32_t t, uint32_t g, uint64_t gmagic, uint32_t (&dig)[D]) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const uint64_t lo = (uint64_t)(uint32_t)gmagic * t;
        const uint64_t hi = (uint64_t)(uint32_t)(gmagic >> 32) * t + (lo >> 32);
        const uint32_t q = (uint32_t)(hi >> 32);
        dig[j] = t - q * g;
        t = q;
    }
}

template <int D>
__device__ __forceinline__ void digits_of(uint64_t t, uint32_t g, uint32_t (&dig)[D]) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
        dig[j] = (uint32_t)(t % (uint64_t)g);
        t /= (uint64_t)g;
    }
}

// Workgroup reduction of the lanes' compensated (I, var) sums: a butterfly in
// each wavefront, then the wavefronts in order.  Thread 0 writes the four
// doubles (sum and compensation of I and var) to out and raises *flag if any
// lane saw a non-finite integrand value.  Ends with a workgroup barrier.
__device__ __forceinline__ void block_totals(double sI, double cI, double sV, double cV, bool bad,
                                             double *out, uint32_t *flag) {
    __shared__ double wave_tot[kMaxBlock / 64][4];
    __shared__ uint32_t wave_bad;
    const int tid = threadIdx.x, nthr = blockDim.x;
    if (tid == 0) wave_bad = 0u;
    __syncthreads();
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const double s2 = __shfl_xor(sI, off, 64), c2 = __shfl_xor(cI, off, 64);
        const double v2 = __shfl_xor(sV, off, 64), e2 = __shfl_xor(cV, off, 64);
        two_sum_merge(sI, cI, s2, c2);
        two_sum_merge(sV, cV, v2, e2);
    }
    const int wave = tid >> 6;
    if ((tid & 63) == 0) {
        wave_tot[wave][0] = sI;
        wave_tot[wave][1] = cI;
        wave_tot[wave][2] = sV;
        wave_tot[wave][3] = cV;
    }
    if (__any(bad) && (tid & 63) == 0) atomicOr(&wave_bad, 1u);
    __syncthreads();
    if (tid == 0) {
        double s0 = wave_tot[0][0], c0 = wave_tot[0][1], v0 = wave_tot[0][2], e0 = wave_tot[0][3];
        for (int wv = 1; wv < nthr / 64; ++wv) {
            two_sum_merge(s0, c0, wave_tot[wv][0], wave_tot[wv][1]);
            two_sum_merge(v0, e0, wave_tot[wv][2], wave_tot[wv][3]);
        }
        out[0] = s0;
        out[1] = c0;
        out[2] = v0;
        out[3] = e0;
        if (wave_bad) atomicOr(flag, 1u);
    }
    __syncthreads();
}

// ---------------------------------------------------------------- the kernel

// One integral: persistent workgroups stride through all m sub-cubes.
// kTraced instantiations additionally write per-sample and per-cube records for
// the sub-cubes [t0, t1); kSplit ones spread the samples of a sub-cube over
// 2^lsplit neighbouring lanes and keep copies of every bin side by side; F32 instantiations evaluate the map and the
// integrand in single precision.  Everything from I_k on is FP64 in both.
template <int F, int D, int KIND, bool F32>
__global__ void __launch_bounds__(kMaxBlock)
    __attribute__((amdgpu_waves_per_eu(kFixedWaves<F, D, KIND, F32> ? kFixedWaves<F, D, KIND, F32> : 1,
                                       kFixedWaves<F, D, KIND, F32> ? kFixedWaves<F, D, KIND, F32> : 8)))
    vsample_kernel(const SampleArgs a) {
    constexpr bool TRACE = KIND == kTraced, FUSED = KIND == kFused, SPLIT = KIND == kSplit || FUSED;
    constexpr bool COPIES = SPLIT || KIND == kCopies;
    constexpr bool J0 = !F32 && (KIND == kPlain || KIND == kCopies);
    constexpr bool LOV = !SPLIT && kLowInVgpr<F, D, F32>;
    if (a.run_last && (int64_t)a.iter > (int64_t)*a.run_last) return;  // the run has ended
    extern __shared__ double lds[];
    const LdsView<F32> v(lds, D, a.nb);
    if constexpr (FUSED) {
        const double *B;
        if (fused::steps<D>(a, v.hist, &B)) return;
        const int nb = a.nb, row = nb + 1;
        if constexpr (F32) {
            const float inv_nb = 1.0f / (float)nb;
            for (int e = threadIdx.x; e < D * nb; e += blockDim.x) {
                const int i = e + fused::row_of(e, inv_nb);  // row j starts j entries later in rows of nb + 1
                v.grid[2 * e] = (float)B[i];
                v.grid[2 * e + 1] = (float)(B[i + 1] - B[i]);
            }
        } else {
            for (int e = threadIdx.x; e < D * row; e += blockDim.x) v.grid[e] = B[e];
        }
        __syncthreads();  // B lies where the histogram will
        if (a.hist)
            for (int i = threadIdx.x; i < D * nb * a.hist_copies; i += blockDim.x) v.hist[i] = 0.0;
    } else {
        load_lds<D, F32>(a, v);
    }
    __syncthreads();
    // the per-axis constants are the same for every lane: read them with
    // scalar loads (constant address space) rather than from LDS, whose
    // bandwidth the grid reads and histogram atomics need.  volatile makes
    // the compiler load each where it is used instead of holding all of them
    // in scalar registers, which spilled them to VGPR lanes and cost a VALU
    // read-back per use.
    volatile Const<real_t<F32>> *sC = (volatile Const<real_t<F32>> *)a.consts;

    // this lane's first sub-cube (below 2^32: at most 2^20 workgroups)
    uint64_t t = ((uint64_t)blockIdx.x * (uint64_t)blockDim.x + (uint64_t)threadIdx.x) >> (SPLIT ? a.lsplit : 0);
    uint32_t dig[D];
    digits_of32<D>((uint32_t)t, (uint32_t)a.g, a.gmagic, dig);
    double sI = 0.0, cI = 0.0, sV = 0.0, cV = 0.0;
    bool bad = false;
    // the lower bounds, copied once into vector registers (the empty asm keeps
    // the copies there rather than reloading them as scalars)
    real_t<F32> lov[D];
    if constexpr (LOV) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            lov[j] = sC[kConstStride * j];
            asm volatile("" : "+v"(lov[j]));
        }
    }
    while (t < (uint64_t)a.m) {
        double It, vt;
        cube_pass<F, D, TRACE, F32, kPairSamples<F, D, F32>, true, LOV, kGridFirst<F, D, F32>,
                  kGridFirst<F, D, F32>, COPIES, SPLIT, 0, false, J0>(a, v, sC, t, dig, It, vt, bad, lov);
        two_sum_add(sI, cI, It);
        two_sum_add(sV, cV, vt);
        // next sub-cube of this lane: t += stride, digit by digit
        t += (uint64_t)a.stride;
        odometer_add<D>(dig, a.sdig, (uint32_t)a.g);
    }
    block_totals(sI, cI, sV, cV, bad, a.partials + 4 * (size_t)blockIdx.x, a.flag);
    if (a.hist) {
        // into accumulator blockIdx % kHistAcc (ordinary device memory, so the
        // hardware FP64 atomic add applies); bins it never reached are skipped
        const int n = D * a.nb;
        double *acc = a.hist_acc + (size_t)(blockIdx.x & ((FUSED ? kFusedAccs : kHistAcc) - 1)) * a.hist_stride;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            double h;
            if constexpr (COPIES) {
                // the copies from a different one on in neighbouring lanes, so
                // that they read different banks
                h = 0.0;
                for (int c = 0; c < a.hist_copies; ++c)
                    h += v.hist[i * a.hist_copies + ((c + (int)threadIdx.x) & (a.hist_copies - 1))];
            } else {
                h = a.hist_copies > 1 ? v.hist[i] + v.hist[n + i] : v.hist[i];
            }
            if (h != 0.0) unsafeAtomicAdd(acc + i, h);
        }
    }
}

// A staged pass of one integral (large adjusting passes): the lattice as g^NS
// blocks of g^K sub-cubes (K = D - NS), a block's sub-cubes in rounds of one per
// lane.  Workgroup b takes the rounds [b T / B, (b + 1) T / B) of the T rounds of
// all blocks, so it walks through one block after another; see SlowAxes.
//
// Bound: VALU issue.  With all axes alike (kPlain, kCopies with 4) the LDS set
// the pace, whose FP64 atomics at random bins cost 26 to 33 cycles per wave
// against 8.7 where no two lanes meet on a bank; here that is so on NS axes, whose
// digits are scalars besides, and on the unit cube (UNIT) the points' scaling,
// an identity there, is left out.  Per pass: d = 8 corner peak, 1e9 samples,
// 500 bins 8310 -> 7450 us (FP64), 5877 -> 4653 (FP32 evaluation); d = 10, 4e8,
// 400 bins 4602 -> 3977 (FP64); d = 9, 8e8, FP32 6415 -> 4980; d = 6 tables, 1e8
// 1004 -> 965 (FP64), 638 -> 594 (FP32); FP64 Gaussian kernels 1.01 to 1.07.
template <int F, int D, int NS, bool F32, bool UNIT>
__global__ void __launch_bounds__(kMaxBlock)
    __attribute__((amdgpu_waves_per_eu(staged_waves(F, D, F32), staged_waves(F, D, F32))))
    vsample_staged_kernel(const SampleArgs a) {
    using R = real_t<F32>;
    constexpr int K = D - NS;
    constexpr bool GF = F32 || kGridFirst<F, D, F32>;
    if (a.run_last && (int64_t)a.iter > (int64_t)*a.run_last) return;  // the run has ended
    extern __shared__ double lds[];
    const int nb = a.nb, row = F32 ? nb : nb + 1, tid = threadIdx.x, nthr = blockDim.x;
    const int W = a.window, wrow = F32 ? W : W + 1;
    LdsView<F32> v(lds, K, nb);
    double *sgrid = v.hist + K * nb * a.hist_copies;  // NS windows of the grid
    double *stage = sgrid + NS * wrow;                // NS windows of copies of the histogram
    load_lds<K, F32>(a, v);
    const int ss = a.stage_shift, quarter = (1 << ss) >> 2;
    for (int i = tid; i < (NS * W) << ss; i += nthr) stage[i] = 0.0;
    volatile Const<R> *sC = (volatile Const<R> *)a.consts;
    constexpr bool LOV = !UNIT && kLowInVgpr<F, D, F32>;
    R lov[D];
    if constexpr (LOV) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            lov[j] = sC[kConstStride * j];
            asm volatile("" : "+v"(lov[j]));
        }
    }
    const uint32_t g = (uint32_t)a.g, C = a.block_cubes, NR = uniform((C + nthr - 1) / nthr);
    const uint64_t T = (uint64_t)a.blocks_total * NR;  // below 2^32 (host)
    uint32_t r = uniform((uint32_t)(T * blockIdx.x / gridDim.x));
    const uint32_t r1 = uniform((uint32_t)(T * (blockIdx.x + 1) / gridDim.x));
    uint32_t sup = uniform(r / NR), rr = r - sup * NR;
    const R s = R(F32 ? a.s32 : a.s);
    double sI = 0.0, cI = 0.0, sV = 0.0, cV = 0.0;
    bool bad = false;
    const uint32_t lane_copy = (uint32_t)(tid & ((1 << ss) - 1)) << 3;
    while (r < r1) {
        SlowAxes<R, NS> slow;
        int i0[NS];
        uint32_t x = sup;
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const uint32_t q = uniform(x / g), c = x - q * g;
            x = q;
            slow.c[j] = uniform(R(c));
            i0[j] = (int)uniform((uint32_t)min((int)(slow.c[j] * s), nb - 1));
            slow.row[j] = lds_address(sgrid + j * wrow) - (uint32_t)i0[j] * 8u;
            slow.stage[j] = lds_address(stage + ((j * W) << ss)) - ((uint32_t)i0[j] << (3 + ss)) + lane_copy;
        }
        // the windows: entries i0 .. i0 + W (FP64: boundaries), beyond the last
        // bin repeated (never read)
        for (int e = tid; e < NS * wrow; e += nthr) {
            const int j = e / wrow, k = e - j * wrow;
            int first = i0[0];
#pragma unroll
            for (int q = 1; q < NS; ++q) first = j == q ? i0[q] : first;
            const double *B = a.grid + (size_t)(K + j) * (nb + 1);
            if constexpr (F32) {
                const int b = min(first + k, nb - 1);
                float2 *cell = reinterpret_cast<float2 *>(sgrid) + e;
                *cell = make_float2((float)B[b], (float)(B[b + 1] - B[b]));
            } else {
                sgrid[e] = B[min(first + k, nb)];
            }
        }
        __syncthreads();
        const uint32_t n = min(NR - rr, r1 - r);
        uint32_t tl = rr * (uint32_t)nthr + (uint32_t)tid;
        uint32_t dig[K];
        digits_of32<K>(tl, g, a.gmagic, dig);
        const uint32_t t0 = sup * C;
        for (uint32_t k = 0; k < n; ++k) {
            if (tl < C) {
                double It, vt;
                cube_pass<F, D, false, F32, false, true, LOV, GF, GF, false, false, NS, UNIT, !F32>(
                    a, v, sC, (uint64_t)(t0 + tl), dig, It, vt, bad, lov, slow);
                two_sum_add(sI, cI, It);
                two_sum_add(sV, cV, vt);
            }
            tl += (uint32_t)nthr;
            odometer_add<K>(dig, a.sdig, g);
        }
        r += n;
        rr = 0;
        ++sup;
        __syncthreads();
        // the windows' sums into the accumulators: four threads per bin, each a
        // quarter of the copies, from a different one on in neighbouring bins
        // (of 32 copies no two lanes of a half-wave then meet on a bank)
        double *acc = a.hist_acc + (size_t)(blockIdx.x % kHistAcc) * a.hist_stride;
        for (int e = tid; e < NS * W * 4; e += nthr) {
            const int bin = e >> 2;
            double h = 0.0, *first_copy = stage + (bin << ss) + (e & 3) * quarter;
            for (int k = 0; k < quarter; ++k) {
                double *q = first_copy + ((k + bin) & (quarter - 1));
                h += *q;
                *q = 0.0;
            }
            h += __shfl_xor(h, 1, 64);
            h += __shfl_xor(h, 2, 64);
            const int j = bin / W;
            int first = i0[0];
#pragma unroll
            for (int q = 1; q < NS; ++q) first = j == q ? i0[q] : first;
            if ((e & 3) == 0 && h != 0.0) unsafeAtomicAdd(acc + (K + j) * nb + first + (bin - j * W), h);
        }
        // (the next block's windows end with a barrier before anything is added)
    }
    block_totals(sI, cI, sV, cV, bad, a.partials + 4 * (size_t)blockIdx.x, a.flag);
    const int n = K * nb;
    double *acc = a.hist_acc + (size_t)(blockIdx.x % kHistAcc) * a.hist_stride;
    for (int i = tid; i < n; i += nthr) {
        const double h = a.hist_copies > 1 ? v.hist[i] + v.hist[n + i] : v.hist[i];
        if (h != 0.0) unsafeAtomicAdd(acc + i, h);
    }
}

template <int F, int D, bool UNIT>
const void *staged_kernel_fd(bool fp32) {
    constexpr int NS = staged_slow_axes(F, D);
    return fp32 ? reinterpret_cast<const void *>(&vsample_staged_kernel<F, D, NS, true, UNIT>)
                : reinterpret_cast<const void *>(&vsample_staged_kernel<F, D, NS, false, UNIT>);
}

// The kernels of one integrand and dimension, as launch_sample takes them.
template <int F, int D>
const void *sample_kernel_fd(int kind, bool fp32) {
    switch (kind) {
    case kStaged:
        if constexpr (staged_slow_axes(F, D) > 0) return staged_kernel_fd<F, D, false>(fp32);
        else return nullptr;
    case kStagedUnit:
        if constexpr (staged_slow_axes(F, D) > 0) return staged_kernel_fd<F, D, true>(fp32);
        else return nullptr;
    case kTraced:
        return fp32 ? reinterpret_cast<const void *>(&vsample_kernel<F, D, kTraced, true>)
                    : reinterpret_cast<const void *>(&vsample_kernel<F, D, kTraced, false>);
    case kPerAxis:
        return fp32 ? nullptr : reinterpret_cast<const void *>(&vsample_kernel<F, D, kPerAxis, false>);
    case kCopies:
        return fp32 ? reinterpret_cast<const void *>(&vsample_kernel<F, D, kCopies, true>)
                    : reinterpret_cast<const void *>(&vsample_kernel<F, D, kCopies, false>);
    case kFused:
        return fp32 ? reinterpret_cast<const void *>(&vsample_kernel<F, D, kFused, true>)
                    : reinterpret_cast<const void *>(&vsample_kernel<F, D, kFused, false>);
    case kSplit:
        return fp32 ? reinterpret_cast<const void *>(&vsample_kernel<F, D, kSplit, true>)
                    : reinterpret_cast<const void *>(&vsample_kernel<F, D, kSplit, false>);
    default:
        return fp32 ? reinterpret_cast<const void *>(&vsample_kernel<F, D, kPlain, true>)
                    : reinterpret_cast<const void *>(&vsample_kernel<F, D, kPlain, false>);
    }
}

}  // namespace mcubes
