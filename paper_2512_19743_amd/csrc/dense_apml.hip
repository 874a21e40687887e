// Dense APML (Sec. III-A): the formulation that sparse APML prunes, kept as a
// baseline. Every pair (i, j) of a sample takes part: no threshold, so the
// plan is the full N x M matrix, for points of any dimension d.
//
//   C_ij = ||x_i - y_j||_2; per row the two smallest costs (decided on the
//   single-precision squared distance, ties to the smaller index), the
//   clamped gap g and the temperature T (Eq. 1); P_row = softmax over the
//   whole row (Eq. 2); the same per column; P0 = (P_row + P_col) / 2;
//   L times column scaling (Eq. 3) then row scaling (Eq. 4); loss = sum P C;
//   the gradient through all of it, temperatures included (Eq. 5 for the
//   distance).
//
// Only P0 is materialised (float32, N x M, rows padded to four). Everything
// else is a per-row or per-column vector, in double precision:
//  * The plan after iteration l is alpha^l_i P0_ij beta^l_j, so a Sinkhorn
//    iteration needs one product of P0 with a column vector and one of its
//    transpose with a row vector. k_dsweep forms both from a single read of P0:
//    a row's product is complete once the row has passed, and the row is then
//    still in registers for the column sums.
//  * The reverse iterations are the recurrences of the sparse path (see the
//    per-iteration reverse launches in sinkhorn.hip), with the same two
//    products per iteration, hence the same kernel; the adjoint of P0 is
//      g alpha^L_i beta^L_j C_ij + sum_l (Rbar^l_i beta^l_j + alpha^(l-1)_i Sbar^l_j),
//    a direct term and a product of two thin matrices of 2L columns, which
//    k_dpair forms on the matrix cores (double precision) for the pairs it
//    holds, never in memory.
//  * C and both softmaxes are recomputed from the coordinates where needed.
// 32 x 2048 x 2048 points, 10 iterations, forward + backward: 26.6 -> 4.3 ms
// against a plan matrix read and written in every half-iteration and a
// double-precision adjoint matrix; bounds by launch: the sweeps read P0 at
// 5.2 TB/s, the others are bound by double-precision arithmetic (a square
// root and one or two exponentials per pair).
//
// Sums have a fixed association: every result is bitwise reproducible.
#include <algorithm>
#include <cmath>

#include "apml_internal.h"
#include "device_common.h"

namespace apml {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// (value, index) is smaller than (v2, i2) in lexicographic order.
__device__ __forceinline__ bool before(float v, int i, float v2, int i2) { return v < v2 || (v == v2 && i < i2); }

// Merges another pair of two smallest (value, index) entries into this one:
// the two smallest of the union multiset, ties to the smaller index.
__device__ __forceinline__ void merge_top2(float &m1, int &k1, float &m2, int &k2, float n1, int q1, float n2,
                                           int q2)
{
    if (before(n1, q1, m1, k1)) {
        // the other list's first is the new first; the second is the smaller
        // of this list's first and the other's second
        if (before(m1, k1, n2, q2)) {
            m2 = m1;
            k2 = k1;
        } else {
            m2 = n2;
            k2 = q2;
        }
        m1 = n1;
        k1 = q1;
    } else if (before(n1, q1, m2, k2)) {
        m2 = n1;
        k2 = q1;
    }
}

// sqrt of a squared distance between float coordinates: 0, or between 1e-90
// and 1e79, so the reciprocal square root needs none of the library's scaling
// (1e-300 is added, below an ulp of any s but 0: its root, 1e-150, is added to
// nothing smaller than 1e-45; a maximum instead would lose a NaN). One
// Goldschmidt step and a residual correction: within an ulp.
__device__ __forceinline__ double root(double s)
{
    s += 1e-300;
    const double y = __builtin_amdgcn_rsq(s);
    double g = s * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    return __builtin_fma(__builtin_fma(-g, g, s), h, g);
}

// 2^t for finite t (above 1024 infinity, below -1100: 0; NaN stays, by f): 2^n (1 + f q(f)), n
// the nearest whole number and |f| <= 1/2, q the polynomial that interpolates (2^f - 1) / f at
// eleven Chebyshev nodes (relative error 2e-17 of 2^f, exactly 1 at 0). 17
// operations against the library exponential's 26, which with the root's 8
// against 19 bound these kernels (32 x 2048 x 2048 points: k_dz 430 -> 319 us,
// k_dp0 335 -> 269, k_dpair 701 -> 589 and 443 -> 388).
__device__ __forceinline__ double exp2_of(double t)
{
    const double w = __builtin_rint(t), n = __builtin_fmax(w, -1100.0), f = t - w;
    double q = 4.4549605981865186e-10;
    q = __builtin_fma(q, f, 7.072585949269223e-09);
    q = __builtin_fma(q, f, 1.0178062445845774e-07);
    q = __builtin_fma(q, f, 1.321544258792169e-06);
    q = __builtin_fma(q, f, 1.525273382983612e-05);
    q = __builtin_fma(q, f, 0.0001540353044173605);
    q = __builtin_fma(q, f, 0.0013333558146416936);
    q = __builtin_fma(q, f, 0.009618129107606888);
    q = __builtin_fma(q, f, 0.0555041086648216);
    q = __builtin_fma(q, f, 0.24022650695910097);
    q = __builtin_fma(q, f, 0.6931471805599453);
    return __builtin_ldexp(__builtin_fma(f, q, 1.0), (int)n);
}

// 1 / v for normal v: the hardware reciprocal and two Newton steps.
__device__ __forceinline__ double inverse(double v)
{
    double r = __builtin_amdgcn_rcp(v);
    r = __builtin_fma(r, __builtin_fma(-v, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-v, r, 1.0), r);
}

// C = ||a - b||_2 in double precision (Sec. III-A).
template <int DP> __device__ __forceinline__ double cost_of(const double (&a)[DP], const double (&b)[DP])
{
    double t = a[0] - b[0];
    double s = t * t;
#pragma unroll
    for (int k = 1; k < DP; ++k) {
        t = a[k] - b[k];
        s = __builtin_fma(t, t, s);
    }
    return root(s);
}

// Softmax entry (Eq. 2) of a pair of cost C for an owner with n2 = -T log2(e), C1 and 1/Z.
__device__ __forceinline__ double softmax_of(double C, double n2, double c1, double iZ)
{
    return exp2_of(n2 * (C - c1)) * iZ;
}

// ---------------------------------------------------------------------------
// coordinates, statistics, normalisers
// ---------------------------------------------------------------------------

// Both clouds with their points padded to DP coordinates (zeros, which add
// nothing to a distance), in single and in double precision.
__global__ __launch_bounds__(kBlock) void k_dprep(DenseDev D)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t nr = (int64_t)D.B * D.N * D.dp, nc = (int64_t)D.B * D.M * D.dp;
    if (t >= nr + nc)
        return;
    const bool rows = t < nr;
    const int64_t e = rows ? t : t - nr, p = e / D.dp;
    const int k = (int)(e - p * D.dp);
    const float v = k < D.d ? (rows ? D.x : D.y)[p * D.d + k] : 0.0f;
    const DenseSide &s = rows ? D.row : D.col;
    s.pf[e] = v;
    s.pd[e] = v;
}

// A launch over the owners of both sides: workgroups of kBlock owners and one
// chunk of the other cloud, the rows' first.
struct Split {
    int blocks_r, blocks_c;   // workgroups per sample and chunk
    int chunks_r, chunks_c;   // chunks of the other cloud
    int len_r, len_c;         // their length
};

struct OwnerBlock {
    bool rows;
    int b, o, chunk, j0, j1; // sample, this lane's owner (may be past the end), the chunk's points
    int n_own, n_oth;
};

__device__ __forceinline__ OwnerBlock owner_block(const DenseDev &D, const Split &s)
{
    OwnerBlock w;
    int g = blockIdx.x;
    const int rows_total = D.B * s.blocks_r * s.chunks_r;
    w.rows = g < rows_total;
    if (!w.rows)
        g -= rows_total;
    const int blocks = w.rows ? s.blocks_r : s.blocks_c, chunks = w.rows ? s.chunks_r : s.chunks_c;
    const int len = w.rows ? s.len_r : s.len_c;
    w.n_own = w.rows ? D.N : D.M;
    w.n_oth = w.rows ? D.M : D.N;
    w.chunk = g % chunks;
    g /= chunks;
    w.o = (g % blocks) * kBlock + (int)threadIdx.x;
    w.b = g / blocks;
    w.j0 = w.chunk * len;
    w.j1 = min(w.n_oth, w.j0 + len);
    return w;
}

// The two nearest points of a chunk of the other cloud per owner, one owner
// per lane, the other points streamed through scalar registers. Bound by its
// issue: about 8 instructions a pair, and the update of the two where some
// lane of the wave meets a smaller distance.
template <int DP> __global__ __launch_bounds__(kBlock) void k_dmin(DenseDev D, Split sp, float4 *part)
{
    const OwnerBlock w = owner_block(D, sp);
    const int o = min(w.o, w.n_own - 1);
    const DenseSide &own = w.rows ? D.row : D.col, &oth = w.rows ? D.col : D.row;
    float a[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k)
        a[k] = own.pf[((size_t)w.b * w.n_own + o) * DP + k];
    const const_ptr<float> q = as_const(oth.pf) + (size_t)w.b * w.n_oth * DP;
    float m1 = kInf, m2 = kInf;
    int k1 = INT_MAX, k2 = INT_MAX;
#pragma unroll 4
    for (int j = w.j0; j < w.j1; ++j) {
        // d0*d0, then fma(dk, dk, s): the sequence of the sparse path's scans
        float t = a[0] - q[(size_t)j * DP];
        float s = t * t;
#pragma unroll
        for (int k = 1; k < DP; ++k) {
            t = a[k] - q[(size_t)j * DP + k];
            s = __builtin_fmaf(t, t, s);
        }
        if (s < m2) {
            if (s < m1) {
                m2 = m1;
                k2 = k1;
                m1 = s;
                k1 = j;
            } else {
                m2 = s;
                k2 = j;
            }
        }
    }
    if (w.o < w.n_own)
        part[(w.rows ? 0 : (size_t)sp.chunks_r * D.B * D.N) +
             (size_t)w.chunk * D.B * w.n_own + (size_t)w.b * w.n_own + o] =
            make_float4(m1, __builtin_bit_cast(float, k1), m2, __builtin_bit_cast(float, k2));
}

// Per owner: the chunks' minima merged, the clamped gap and the temperature
// (Eq. 1); the scalings before the first iteration are 1.
template <int DP>
__global__ __launch_bounds__(kBlock) void k_dstat(DenseDev D, Split sp, const float4 *part, double lk_row, double lk_col)
{
    const int BN = D.B * D.N, BM = D.B * D.M;
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= BN + BM)
        return;
    const bool rows = t < BN;
    const int o = rows ? t : t - BN, n_own = rows ? D.N : D.M, n_oth = rows ? D.M : D.N, b = o / n_own;
    const DenseSide &s = rows ? D.row : D.col, &oth = rows ? D.col : D.row;
    if (!rows)
        part += (size_t)sp.chunks_r * BN;
    float m1 = kInf, m2 = kInf;
    int k1 = INT_MAX, k2 = INT_MAX;
    for (int c = 0; c < (rows ? sp.chunks_r : sp.chunks_c); ++c) {
        const float4 v = part[(size_t)c * (rows ? BN : BM) + o];
        merge_top2(m1, k1, m2, k2, v.x, __builtin_bit_cast(int, v.y), v.z, __builtin_bit_cast(int, v.w));
    }
    // only distances that overflow single precision leave an index unset
    if (k1 == INT_MAX)
        k1 = 0;
    if (k2 == INT_MAX || k2 == k1)
        k2 = k1 == 0 ? 1 : 0;
    double a[DP], p[DP], q[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k) {
        a[k] = s.pd[(size_t)o * DP + k];
        p[k] = oth.pd[((size_t)b * n_oth + k1) * DP + k];
        q[k] = oth.pd[((size_t)b * n_oth + k2) * DP + k];
    }
    const double c1 = cost_of(a, p), c2 = cost_of(a, q);
    const double gap = (c2 - c1) + D.delta;
    const bool clamped = gap < D.eps_gap;
    const double g = clamped ? D.eps_gap : gap;
    s.k1[o] = k1;
    s.k2[o] = k2;
    s.c1[o] = c1;
    s.g[o] = g;
    s.T[o] = (rows ? lk_row : lk_col) / g;
    // a T beyond 1e250 (a clamped gap of a tiny eps_gap) as 1e250: every difference of
    // costs but 0 gives the same 0 or infinity, and the product stays finite (exp2_of)
    const double n2 = -1.4426950408889634 * s.T[o];
    s.n2[o] = n2 < -1e250 && n2 >= -1.7976931348623157e308 ? -1e250 : n2;
    s.clamped[o] = clamped;
    s.sc[o] = 1.0;
}

// Softmax normalisers over a chunk, Z = sum exp(-T (C - C1)) (Eq. 2), one
// owner per lane, the other points through scalar registers.
template <int DP> __global__ __launch_bounds__(kBlock) void k_dz(DenseDev D, Split sp, double *part)
{
    const OwnerBlock w = owner_block(D, sp);
    const int o = min(w.o, w.n_own - 1);
    const DenseSide &own = w.rows ? D.row : D.col, &oth = w.rows ? D.col : D.row;
    const size_t go = (size_t)w.b * w.n_own + o;
    double a[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k)
        a[k] = own.pd[go * DP + k];
    const double n2 = own.n2[go], c1 = own.c1[go];
    const const_ptr<double> q = as_const(oth.pd) + (size_t)w.b * w.n_oth * DP;
    double z = 0.0;
#pragma unroll 2
    for (int j = w.j0; j < w.j1; ++j) {
        double p[DP];
#pragma unroll
        for (int k = 0; k < DP; ++k)
            p[k] = q[(size_t)j * DP + k];
        z += exp2_of(n2 * (cost_of(a, p) - c1));
    }
    if (w.o < w.n_own)
        part[(w.rows ? 0 : (size_t)sp.chunks_r * D.B * D.N) + (size_t)w.chunk * D.B * w.n_own + go] = z;
}

// 1/Z per owner from the chunks' sums.
__global__ __launch_bounds__(kBlock) void k_dzsum(DenseDev D, Split sp, const double *part)
{
    const int BN = D.B * D.N, BM = D.B * D.M;
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= BN + BM)
        return;
    const bool rows = t < BN;
    const int o = rows ? t : t - BN, n = rows ? BN : BM;
    if (!rows)
        part += (size_t)sp.chunks_r * BN;
    double z = 0.0;
    for (int c = 0; c < (rows ? sp.chunks_r : sp.chunks_c); ++c)
        z += part[(size_t)c * n + o];
    (rows ? D.row : D.col).iZ[o] = 1.0 / z;
}

// P0 = (P_row + P_col) / 2 (Sec. III-A) of one chunk of rows, one column per
// lane, the rows' values through scalar registers, and the chunk's column
// sums (Eq. 3 of the first iteration). Padding columns hold 0.
template <int DP> __global__ __launch_bounds__(kBlock) void k_dp0(DenseDev D, int rows_per, int chunks, double *part)
{
    const int col_blocks = (D.ld + kBlock - 1) / kBlock;
    int g = blockIdx.x;
    const int jb = g % col_blocks;
    g /= col_blocks;
    const int ch = g % chunks, b = g / chunks;
    const int j = jb * kBlock + (int)threadIdx.x;
    const int i0 = ch * rows_per, i1 = min(D.N, i0 + rows_per);
    const size_t c = (size_t)b * D.M + min(j, D.M - 1);
    double a[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k)
        a[k] = D.col.pd[c * DP + k];
    const double n2 = D.col.n2[c], c1 = D.col.c1[c], iZ = j < D.M ? D.col.iZ[c] : 0.0;
    const const_ptr<double> q = as_const(D.row.pd) + (size_t)b * D.N * DP;
    const const_ptr<double> rn2 = as_const(D.row.n2) + (size_t)b * D.N, rc1 = as_const(D.row.c1) + (size_t)b * D.N,
                            rZ = as_const(D.row.iZ) + (size_t)b * D.N;
    float *out = D.P0 + ((size_t)b * D.N) * D.ld + j;
    double sum = 0.0;
    for (int i = i0; i < i1; ++i) {
        double p[DP];
#pragma unroll
        for (int k = 0; k < DP; ++k)
            p[k] = q[(size_t)i * DP + k];
        const double C = cost_of(a, p);
        const float p0 = (float)(0.5 * (softmax_of(C, rn2[i], rc1[i], rZ[i]) + softmax_of(C, n2, c1, iZ)));
        const float v = j < D.M ? p0 : 0.0f;
        if (j < D.ld)
            out[(size_t)i * D.ld] = v;
        sum += (double)v;
    }
    if (j < D.ld)
        part[((size_t)b * chunks + ch) * D.ld + j] = sum;
}

// ---------------------------------------------------------------------------
// Sinkhorn iterations, forward and reverse
// ---------------------------------------------------------------------------

// With N != M the unit marginals cannot both hold: alpha grows and beta
// shrinks by about N / M in every iteration. The stored scalings are
// a^l = alpha^l 2^(-e_l) and c^l = beta^l 2^(e_(l-1)), e_l = round(l log2(N / M)),
// so that any number of iterations stays in range; the products that the
// plan and its adjoint need carry no factor (the last iteration takes e_L =
// e_(L-1)). f_in and f_out below are the powers of two between the steps.
enum DenseMode { FWD, BWD };

// One launch: iteration l forward, or its reverse.
//   FWD: c^l from the column sums in part_in (or already there), the rows'
//        products with it, a^l, and the column sums of a^l P0 into part_out.
//   BWD: Sbar^l from the sums in part_in, the rows' products with it,
//        Rbar^(l-1), and the column sums of Rbar^(l-1) P0.
struct Sweep {
    const double *part_in; // [B][parts][ld]
    double *part_out;      // [B][nb][ld], or NULL
    int parts;             // partial sums per column; 0: the column values are in memory
    int nb, rb;            // row blocks per sample and rows per block
    int l, b0;             // iteration; first sample of the launch
    double f_in, f_out;
};

template <DenseMode MODE>
__device__ __forceinline__ double column_value(const DenseDev &D, const Sweep &s, size_t c, double sum)
{
    const size_t BM = (size_t)D.B * D.M;
    if constexpr (MODE == FWD) {
        const double prev = D.col.sc[(size_t)(s.l - 1) * BM + c] * s.f_in;
        return prev * inverse(prev * sum + D.eps_stab);
    } else {
        const double cl = D.col.sc[(size_t)s.l * BM + c];
        const double old = s.l < D.L ? s.f_in * D.col.sb[(size_t)s.l * BM + c] : 0.0;
        return old - cl * cl * sum;
    }
}

// Where the column values of a launch live.
template <DenseMode MODE> __device__ __forceinline__ double *column_slot(const DenseDev &D, int l)
{
    const size_t BM = (size_t)D.B * D.M;
    return MODE == FWD ? D.col.sc + (size_t)l * BM : D.col.sb + (size_t)(l - 1) * BM;
}

// What a row's new value needs besides its product, and the value.
struct RowOld {
    double a, r;
};
template <DenseMode MODE> __device__ __forceinline__ RowOld row_old(const DenseDev &D, const Sweep &s, size_t r)
{
    const size_t BN = (size_t)D.B * D.N;
    return {D.row.sc[(size_t)(s.l - 1) * BN + r], MODE == BWD ? D.row.sb[(size_t)(s.l - 1) * BN + r] : 0.0};
}
template <DenseMode MODE>
__device__ __forceinline__ double row_value(const DenseDev &D, const Sweep &s, const RowOld &o, double dot)
{
    if constexpr (MODE == FWD)
        return o.a * inverse(o.a * dot + D.eps_stab) * s.f_out;
    else
        return s.f_out * (D.eps_stab * o.r - o.a * o.a * dot);
}
template <DenseMode MODE> __device__ __forceinline__ double *row_slot(const DenseDev &D, int l)
{
    const size_t BN = (size_t)D.B * D.N;
    return MODE == FWD ? D.row.sc + (size_t)l * BN : D.row.sb + (size_t)(l - 2) * BN;
}

// v rotated by N lanes within each row of 16.
template <int N> __device__ __forceinline__ double row_ror(double v)
{
    int2 w = __builtin_bit_cast(int2, v);
    w.x = __builtin_amdgcn_update_dpp(0, w.x, 0x120 + N, 0xF, 0xF, true);
    w.y = __builtin_amdgcn_update_dpp(0, w.y, 0x120 + N, 0xF, 0xF, true);
    return __builtin_bit_cast(double, w);
}

// Sums of four values at once over each row of 16 lanes: lane l returns that
// of v[l % 4]. Two exchanges halve the values a lane holds, so that four sums
// cost little more than one.
__device__ __forceinline__ double row_sum4(const double (&v)[4])
{
    const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
    const double lo = (b0 ? v[1] : v[0]) + partner<0>(b0 ? v[0] : v[1]);
    const double hi = (b0 ? v[3] : v[2]) + partner<0>(b0 ? v[2] : v[3]);
    double s = (b1 ? hi : lo) + partner<1>(b1 ? lo : hi);
    s += row_ror<4>(s);
    s += row_ror<8>(s);
    return s;
}

// And over the wave.
__device__ __forceinline__ double wave_sum4(const double (&v)[4])
{
    double s = row_sum4(v);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    return s;
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const int2 w = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(
        double, make_int2(__builtin_amdgcn_readlane(w.x, lane), __builtin_amdgcn_readlane(w.y, lane)));
}

// One iteration from one read of P0: a workgroup of W waves takes rb rows of a
// sample, each lane 4 Q columns, four rows at a time with the next four in
// flight: their products with the column values (v, in registers), summed over
// the workgroup, the rows' new values, then the rows, still in registers, into
// the lane's column sums. W and Q by the row length: M <= 256 W Q, so that a
// row is in registers once (Q = 2 at most: 128 registers a lane at W = 16).
// Bound by the read of P0.
template <DenseMode MODE, int W, int Q> __global__ __launch_bounds__(64 * W) void k_dsweep(DenseDev D, Sweep s)
{
    constexpr int T = 64 * W;
    constexpr int AHEAD = W == 16 ? 0 : 1; // row groups in flight ahead (none fit the 128 registers at 16 waves)
    constexpr int SUMS = W == 1 ? 0 : W <= 4 ? 4 : 1; // sums a wave leaves in LDS per row: of its rows of 16 lanes, or one
    __shared__ double sums[2][W * (SUMS ? SUMS : 1)][4];
    const int g = xcd_contiguous(blockIdx.x, gridDim.x); // a sample's blocks share an L2
    const int b = s.b0 + g / s.nb, blk = g % s.nb;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int r0 = blk * s.rb, r1 = min(D.N, r0 + s.rb);
    const size_t col0 = (size_t)b * D.M, row0 = (size_t)b * D.N;
    const int ld4 = D.ld / 4;
    double v[Q][4], acc[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int j4 = q * T + tid;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            v[q][k] = acc[q][k] = 0.0;
        if (j4 < ld4) {
            if (s.parts) {
                const double2 *in = reinterpret_cast<const double2 *>(s.part_in + (size_t)b * s.parts * D.ld) + 2 * j4;
                double2 lo = make_double2(0.0, 0.0), hi = lo;
#pragma unroll 4
                for (int p = 0; p < s.parts; ++p) {
                    const double2 a = in[(size_t)p * (D.ld / 2)], c = in[(size_t)p * (D.ld / 2) + 1];
                    lo.x += a.x;
                    lo.y += a.y;
                    hi.x += c.x;
                    hi.y += c.y;
                }
                const double sum[4] = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (4 * j4 + k < D.M) {
                        v[q][k] = column_value<MODE>(D, s, col0 + 4 * j4 + k, sum[k]);
                        if (blk == 0)
                            column_slot<MODE>(D, s.l)[col0 + 4 * j4 + k] = v[q][k];
                    }
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (4 * j4 + k < D.M)
                        v[q][k] = column_slot<MODE>(D, s.l)[col0 + 4 * j4 + k];
            }
        }
    }
    const float4 *P = reinterpret_cast<const float4 *>(D.P0 + row0 * D.ld);
    auto load = [&](float4 (&p)[4][Q], int r) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int j4 = q * T + tid;
                p[k][q] = j4 < ld4 ? P[(size_t)min(r + k, r1 - 1) * ld4 + j4] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
    };
    auto old_of = [&](int r) { return row_old<MODE>(D, s, row0 + min(r + (lane & 3), r1 - 1)); };
    float4 p[4][Q], ahead[AHEAD ? AHEAD : 1][4][Q];
    load(p, r0);
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        load(ahead[a], r0 + 4 * (a + 1)); // past the block: its last row again
    RowOld old_next = old_of(r0);
    int par = 0;
    for (int r = r0; r < r1; r += 4, par ^= 1) {
        const RowOld old = old_next;
        old_next = old_of(r + 4);
        float4 last[4][Q];
        if constexpr (AHEAD > 0)
            load(last, r + 4 * (AHEAD + 1));
        double dot[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            dot[k] = 0.0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                dot[k] = __builtin_fma((double)p[k][q].x, v[q][0], dot[k]);
                dot[k] = __builtin_fma((double)p[k][q].y, v[q][1], dot[k]);
                dot[k] = __builtin_fma((double)p[k][q].z, v[q][2], dot[k]);
                dot[k] = __builtin_fma((double)p[k][q].w, v[q][3], dot[k]);
            }
        }
        double t = SUMS == 4 ? row_sum4(dot) : wave_sum4(dot);
        if constexpr (SUMS > 0) {
            if ((lane & (64 / SUMS - 1)) < 4)
                sums[par][wave * SUMS + (SUMS == 4 ? lane >> 4 : 0)][lane & 3] = t; // the other half is still read
            lds_barrier();
            double part[4] = {};
#pragma unroll
            for (int w = 0; w < W * SUMS; ++w)
                part[w & 3] += sums[par][w][lane & 3];
            t = (part[0] + part[1]) + (part[2] + part[3]);
        }
        const double w = row_value<MODE>(D, s, old, t);
        if (wave == 0 && lane < 4 && r + lane < r1)
            row_slot<MODE>(D, s.l)[row0 + r + lane] = w;
        if (s.part_out) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double wk = r + k < r1 ? lane_value(w, k) : 0.0;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    acc[q][0] = __builtin_fma(wk, (double)p[k][q].x, acc[q][0]);
                    acc[q][1] = __builtin_fma(wk, (double)p[k][q].y, acc[q][1]);
                    acc[q][2] = __builtin_fma(wk, (double)p[k][q].z, acc[q][2]);
                    acc[q][3] = __builtin_fma(wk, (double)p[k][q].w, acc[q][3]);
                }
            }
        }
        if constexpr (AHEAD > 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    p[k][q] = ahead[0][k][q];
#pragma unroll
                    for (int a = 0; a + 1 < AHEAD; ++a)
                        ahead[a][k][q] = ahead[a + 1][k][q];
                    ahead[AHEAD - 1][k][q] = last[k][q];
                }
        } else {
            load(p, r + 4);
        }
    }
    if (s.part_out) {
        double2 *out = reinterpret_cast<double2 *>(s.part_out + ((size_t)b * s.nb + blk) * D.ld);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int j4 = q * T + tid;
            if (j4 < ld4) {
                out[2 * j4] = make_double2(acc[q][0], acc[q][1]);
                out[2 * j4 + 1] = make_double2(acc[q][2], acc[q][3]);
            }
        }
    }
}

// The column values of a launch from many partial sums (one column per thread).
template <DenseMode MODE> __global__ __launch_bounds__(kBlock) void k_dcolumns(DenseDev D, Sweep s)
{
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= (int64_t)D.B * D.M)
        return;
    const int b = (int)(c / D.M), j = (int)(c - (int64_t)b * D.M);
    const double *in = s.part_in + (size_t)b * s.parts * D.ld + j;
    double sum = 0.0;
#pragma unroll 8
    for (int p = 0; p < s.parts; ++p)
        sum += in[(size_t)p * D.ld];
    column_slot<MODE>(D, s.l)[c] = column_value<MODE>(D, s, c, sum);
}

// Row products over longer rows, four rows per wave: FWD and BWD as in
// k_dsweep; ROW_LOSS: sum_j P0_ij c^L_j C_ij, the row's share of the loss.
enum RowOp { ROW_FWD, ROW_BWD, ROW_LOSS };

template <int OP, int DP> __global__ __launch_bounds__(kBlock) void k_drow(DenseDev D, Sweep s)
{
    const int row_groups = (D.N + 3) / 4;
    const int64_t g = (int64_t)xcd_contiguous(blockIdx.x, gridDim.x) * (kBlock / 64) + (threadIdx.x >> 6);
    if (g >= (int64_t)D.B * row_groups)
        return;
    const int b = (int)(g / row_groups), r = (int)(g - (int64_t)b * row_groups) * 4, lane = lane_id();
    const size_t row0 = (size_t)b * D.N, col0 = (size_t)b * D.M;
    const double *v = OP == ROW_LOSS ? D.col.sc + (size_t)D.L * D.B * D.M
                                     : column_slot<OP == ROW_BWD ? BWD : FWD>(D, s.l);
    const float *P[4];
    double x[4][DP];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = __builtin_amdgcn_readfirstlane(min(r + k, D.N - 1));
        P[k] = D.P0 + (row0 + i) * D.ld;
#pragma unroll
        for (int e = 0; e < DP; ++e)
            x[k][e] = OP == ROW_LOSS ? as_const(D.row.pd)[(row0 + i) * DP + e] : 0.0;
    }
    double dot[4] = {};
#pragma unroll 2
    for (int j = lane; j < D.M; j += 64) {
        const double vj = v[col0 + j];
        double y[DP];
        if constexpr (OP == ROW_LOSS) {
#pragma unroll
            for (int e = 0; e < DP; ++e)
                y[e] = D.col.pd[(col0 + j) * DP + e];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double pv = (double)P[k][j] * vj;
            if constexpr (OP == ROW_LOSS)
                pv *= cost_of(x[k], y);
            dot[k] += pv;
        }
    }
    const double t = wave_sum4(dot);
    if (lane < 4 && r + lane < D.N) {
        const size_t i = row0 + r + lane;
        if constexpr (OP == ROW_LOSS) {
            D.rowc[i] = t;
        } else {
            constexpr DenseMode M = OP == ROW_BWD ? BWD : FWD;
            row_slot<M>(D, s.l)[i] = row_value<M>(D, s, row_old<M>(D, s, i), t);
        }
    }
}

// Column sums over a block of rows, one column per lane, the rows' values
// through scalar registers: COL_W: sum_i w_i P0_ij; COL_DIRECT: sum_i (g a^L_i
// C_ij + Rbar^L_i) P0_ij, from which Sbar^L follows.
enum ColOp { COL_W, COL_DIRECT };

template <int OP, int DP> __global__ __launch_bounds__(kBlock) void k_dcol(DenseDev D, Sweep s, const double *w)
{
    const int col_blocks = (D.ld + kBlock - 1) / kBlock;
    int g = xcd_contiguous(blockIdx.x, gridDim.x);
    const int jb = g % col_blocks;
    g /= col_blocks;
    const int blk = g % s.nb, b = g / s.nb;
    const int j = min(jb * kBlock + (int)threadIdx.x, D.ld - 1);
    const int i0 = blk * s.rb, i1 = min(D.N, i0 + s.rb);
    const size_t row0 = (size_t)b * D.N;
    const const_ptr<double> wr = as_const(w) + row0;
    const const_ptr<double> ar = as_const(D.row.sc) + (size_t)D.L * D.B * D.N + row0, xr = as_const(D.row.pd) + row0 * DP;
    const double gl = OP == COL_DIRECT ? (double)D.grad_loss[b] : 0.0;
    double y[DP];
    if constexpr (OP == COL_DIRECT) {
#pragma unroll
        for (int e = 0; e < DP; ++e)
            y[e] = D.col.pd[((size_t)b * D.M + min(j, D.M - 1)) * DP + e];
    }
    const float *P = D.P0 + row0 * D.ld + j;
    double acc = 0.0;
#pragma unroll 4
    for (int i = i0; i < i1; ++i) {
        double f = wr[i];
        if constexpr (OP == COL_DIRECT) {
            double x[DP];
#pragma unroll
            for (int e = 0; e < DP; ++e)
                x[e] = xr[(size_t)i * DP + e];
            f = __builtin_fma(gl * ar[i], cost_of(y, x), f);
        }
        acc = __builtin_fma(f, (double)P[(size_t)i * D.ld], acc);
    }
    if (jb * kBlock + (int)threadIdx.x < D.ld)
        s.part_out[((size_t)b * s.nb + blk) * D.ld + j] = acc;
}

// loss_b = sum_i a^L_i sum_j P0_ij c^L_j C_ij (Sec. III-D).
__global__ __launch_bounds__(kBlock) void k_dloss_sum(DenseDev D)
{
    __shared__ double part[kBlock / 64];
    const int b = blockIdx.x;
    const double *a = D.row.sc + (size_t)D.L * D.B * D.N + (size_t)b * D.N, *c = D.rowc + (size_t)b * D.N;
    double acc = 0.0;
    for (int i = threadIdx.x; i < D.N; i += kBlock)
        acc = __builtin_fma(a[i], c[i], acc);
    acc = wave_sum(acc);
    if (lane_id() == 0)
        part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kBlock / 64; ++w)
            s += part[w];
        D.loss[b] = (float)s;
    }
}

// Rbar^L_i = -(a^L_i)^2 g sum_j P0_ij c^L_j C_ij.
__global__ __launch_bounds__(kBlock) void k_drbar(DenseDev D)
{
    const int64_t BN = (int64_t)D.B * D.N, r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= BN)
        return;
    const double a = D.row.sc[(size_t)D.L * BN + r];
    D.row.sb[(size_t)(D.L - 1) * BN + r] = -(a * a) * ((double)D.grad_loss[r / D.N] * D.rowc[r]);
}

// ---------------------------------------------------------------------------
// softmax and distance adjoints
// ---------------------------------------------------------------------------

// Sums over a chunk of the other cloud for 64 owners of one side (16 per
// wave), from the adjoint of P0 of every pair, Pbar.
//   sums (GRAD = false), half = Pbar / 2, P the owner's softmax:
//     sum P half (sigma), sum P half (C - C1), sum P (C - C1)
//   gradient (GRAD = true): with cbar the cost adjoint of the pair (the direct
//     term grad_loss v, both softmax adjoints -T P (half - sigma), the gap term
//     of the other point where this owner is one of its minima),
//     sum cbar / (C + eps_dist) (own - other)     (Eq. 5)
// The product of thin matrices in Pbar is formed on the matrix cores for 16
// others x 16 owners at a time, kKC of its 2L columns a step: up to 16
// iterations the owners' columns stay in registers and the others' are staged
// once per 64 others in LDS, shared by the waves. Lane l then holds owner l %
// 16 and the others l / 16 + 4 r, and does their exponentials and square
// roots, which bound the kernel.
constexpr int kKC = 32;     // columns of the thin matrices per step
constexpr int kPairT = 64;  // others per step
constexpr int kUP = kPairT + 16; // LDS pitch: the four k of an operand in different banks

template <int DP, bool GRAD> struct PairLds {
    double u[kKC][kUP];
    double xyz[kPairT][DP];
    double dir[kPairT];
    double nT[GRAD ? kPairT : 1], n2[GRAD ? kPairT : 1], c1[GRAD ? kPairT : 1], iZ[GRAD ? kPairT : 1], sig[GRAD ? kPairT : 1];
    int2 k12[GRAD ? kPairT : 1];
};

// Column k of a side's thin matrix: the pairs (Rbar^l_i, beta^l_j) at even k,
// (alpha^(l-1)_i, Sbar^l_j) at odd k, l = k / 2 + 1.
template <bool ROWS> __device__ __forceinline__ const double *thin_column(const DenseDev &D, int k)
{
    const DenseSide &s = ROWS ? D.row : D.col;
    const size_t n = (size_t)D.B * (ROWS ? D.N : D.M);
    const int it = k >> 1;
    if (ROWS)
        return (k & 1) ? s.sc + it * n : s.sb + it * n;
    return (k & 1) ? s.sb + it * n : s.sc + (it + 1) * n;
}

template <int DP, bool ROWS, bool GRAD>
__global__ __launch_bounds__(kBlock, DP <= 4 ? 4 : 2) void k_dpair(DenseDev D, int tiles, int chunks, int len, double *part)
{
    constexpr int NV = GRAD ? DP : 3;
    __shared__ PairLds<DP, GRAD> sh;
    const DenseSide &own = ROWS ? D.row : D.col, &oth = ROWS ? D.col : D.row;
    const int n_own = ROWS ? D.N : D.M, n_oth = ROWS ? D.M : D.N;
    int g = xcd_contiguous(blockIdx.x, gridDim.x);
    const int ch = g % chunks;
    g /= chunks;
    const int tile = g % tiles, b = g / tiles;
    const int tid = threadIdx.x, lane = lane_id(), lo = lane & 15, hi = lane >> 4;
    const int o = tile * 64 + (tid >> 6) * 16 + lo;
    const size_t own0 = (size_t)b * n_own, oth0 = (size_t)b * n_oth, po = own0 + min(o, n_own - 1);
    const int j0 = ch * len, j1 = min(n_oth, j0 + len);
    const int K = 2 * D.L;
    const double gl = D.grad_loss[b];
    double a[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k)
        a[k] = own.pd[po * DP + k];
    const double nT = -own.T[po], n2 = own.n2[po], c1 = own.c1[po], iZ = own.iZ[po];
    const double sig = GRAD ? own.sigma[po] : 0.0;
    const double dir = own.sc[(size_t)D.L * D.B * n_own + po];
    double bop[kKC / 4]; // this lane's owner values of a step's columns k = 4 s + l / 16
    auto owner_columns = [&](int kc) {
#pragma unroll
        for (int s = 0; s < kKC / 4; ++s) {
            const int k = kc + 4 * s + hi;
            bop[s] = k < K ? thin_column<ROWS>(D, k)[po] : 0.0;
        }
    };
    if (K <= kKC)
        owner_columns(0);
    double acc[NV] = {};
    for (int t0 = j0; t0 < j1; t0 += kPairT) {
        const int cnt = min(kPairT, j1 - t0);
        __syncthreads(); // the previous step's values are still read
        for (int e = tid; e < kPairT * DP; e += kBlock)
            sh.xyz[e / DP][e % DP] = oth.pd[(oth0 + t0 + min(e / DP, cnt - 1)) * DP + e % DP];
        if (tid < kPairT) {
            const size_t q = oth0 + t0 + min(tid, cnt - 1);
            sh.dir[tid] = oth.sc[(size_t)D.L * D.B * n_oth + q];
            if constexpr (GRAD) {
                sh.nT[tid] = -oth.T[q];
                sh.n2[tid] = oth.n2[q];
                sh.c1[tid] = oth.c1[q];
                sh.iZ[tid] = oth.iZ[q];
                sh.sig[tid] = oth.sigma[q];
                sh.k12[tid] = make_int2(oth.k1[q], oth.k2[q]);
            }
        }
        if (K <= kKC) {
            int row = tid >> 6, i = tid & 63;
            asm volatile("" : "+v"(row)); // the addresses formed here again, not held across the steps
            for (int k = row; k < (K + 3 & ~3); k += kBlock / 64) // 0 from K up to a multiple of 4
                sh.u[k][i] = k < K ? thin_column<!ROWS>(D, k)[oth0 + t0 + min(i, cnt - 1)] : 0.0;
        }
        __syncthreads();
#pragma unroll 1
        for (int t = 0; t < kPairT / 16; ++t) {
            f64x4 pb = {};
            if (K <= kKC) {
#pragma unroll
                for (int s = 0; s < kKC / 4; ++s)
                    if (4 * s < K)
                        pb = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.u[4 * s + hi][t * 16 + lo], bop[s], pb, 0, 0, 0);
            } else {
                for (int kc = 0; kc < K; kc += kKC) {
                    __syncthreads();
                    for (int k = tid >> 4; k < kKC; k += kBlock / 16)
                        sh.u[k][tid & 15] =
                            kc + k < K ? thin_column<!ROWS>(D, kc + k)[oth0 + t0 + min(t * 16 + (tid & 15), cnt - 1)]
                                       : 0.0;
                    owner_columns(kc);
                    __syncthreads();
#pragma unroll
                    for (int s = 0; s < kKC / 4; ++s)
                        pb = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.u[4 * s + hi][lo], bop[s], pb, 0, 0, 0);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = t * 16 + hi + 4 * r;
                double u[DP], q = 0.0;
#pragma unroll
                for (int k = 0; k < DP; ++k) {
                    u[k] = a[k] - sh.xyz[i][k];
                    q = k == 0 ? u[k] * u[k] : __builtin_fma(u[k], u[k], q);
                }
                const double C = root(q);
                const double v = dir * sh.dir[i]; // alpha^L beta^L
                const double half = 0.5 * __builtin_fma(gl * v, C, pb[r]);
                const double e = C - c1;
                double p = exp2_of(n2 * e) * iZ;
                if constexpr (!GRAD) {
                    p = i < cnt ? p : 0.0;
                    const double ph = p * half;
                    acc[0] += ph;
                    acc[1] = __builtin_fma(ph, e, acc[1]);
                    acc[2] = __builtin_fma(p, e, acc[2]);
                } else {
                    const double po_ = softmax_of(C, sh.n2[i], sh.c1[i], sh.iZ[i]);
                    const float p0 = (float)(0.5 * (p + po_));
                    double cb = gl * ((double)p0 * v);
                    cb = __builtin_fma(nT * p, half - sig, cb);
                    cb = __builtin_fma(sh.nT[i] * po_, half - sh.sig[i], cb);
                    const int2 k12 = sh.k12[i];
                    if (o == k12.x || o == k12.y) { // the other point's gap term
                        const double gb = oth.gbar[oth0 + t0 + min(i, cnt - 1)];
                        if (o == k12.y)
                            cb += gb;
                        if (o == k12.x)
                            cb -= gb;
                    }
                    const double w = i < cnt ? cb * inverse(C + D.eps_dist) : 0.0;
#pragma unroll
                    for (int k = 0; k < DP; ++k)
                        acc[k] = __builtin_fma(w, u[k], acc[k]);
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        acc[k] += __shfl_xor(acc[k], 16);
        acc[k] += __shfl_xor(acc[k], 32);
    }
    if (lane < 16 && o < n_own) {
#pragma unroll
        for (int k = 0; k < NV; ++k)
            part[((size_t)ch * D.B * n_own + po) * NV + k] = acc[k];
    }
}

// Per owner: sigma = sum P half, the temperature adjoint Tbar = -sum P (half -
// sigma)(C - C1) and the gap adjoint -Tbar T / g of an unclamped owner.
__global__ __launch_bounds__(kBlock) void k_dsigma(DenseDev D, int rows, int chunks, const double *part)
{
    const int64_t n = (int64_t)D.B * (rows ? D.N : D.M), o = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (o >= n)
        return;
    double s[3] = {};
    for (int c = 0; c < chunks; ++c)
        for (int k = 0; k < 3; ++k)
            s[k] += part[((size_t)c * n + o) * 3 + k];
    const DenseSide &d = rows ? D.row : D.col;
    const double tbar = s[0] * s[2] - s[1];
    d.sigma[o] = s[0];
    d.gbar[o] = (D.tgrad_full && !d.clamped[o]) ? -tbar * d.T[o] / d.g[o] : 0.0;
}

// The gradient of one side: the chunks' sums and the owner's own gap terms.
template <int DP> __global__ __launch_bounds__(kBlock) void k_dgrad(DenseDev D, int rows, int chunks, const double *part)
{
    const int n_own = rows ? D.N : D.M, n_oth = rows ? D.M : D.N;
    const int64_t n = (int64_t)D.B * n_own, o = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (o >= n)
        return;
    const DenseSide &own = rows ? D.row : D.col, &oth = rows ? D.col : D.row;
    const size_t oth0 = (size_t)(o / n_own) * n_oth;
    double acc[DP] = {};
    for (int c = 0; c < chunks; ++c)
#pragma unroll
        for (int k = 0; k < DP; ++k)
            acc[k] += part[((size_t)c * n + o) * DP + k];
    const double gb = own.gbar[o];
    if (gb != 0.0) {
        double a[DP], p[DP], q[DP];
#pragma unroll
        for (int k = 0; k < DP; ++k) {
            a[k] = own.pd[o * DP + k];
            p[k] = oth.pd[(oth0 + own.k1[o]) * DP + k];
            q[k] = oth.pd[(oth0 + own.k2[o]) * DP + k];
        }
        const double w1 = -gb / (cost_of(a, p) + D.eps_dist), w2 = gb / (cost_of(a, q) + D.eps_dist);
#pragma unroll
        for (int k = 0; k < DP; ++k)
            acc[k] += w2 * (a[k] - q[k]) + w1 * (a[k] - p[k]);
    }
    float *out = (rows ? D.grad_x : D.grad_y) + o * D.d;
#pragma unroll
    for (int k = 0; k < DP; ++k)
        if (k < D.d)
            out[k] = (float)acc[k];
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------

int ceil_to(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Chunks of n_oth points for `blocks` workgroups of each, so that about
// `target` run: at least `least` points a chunk, a multiple of `unit`.
void chunk_up(int64_t blocks, int n_oth, int target, int least, int unit, int *chunks, int *len)
{
    const int64_t want = std::max<int64_t>(1, (target + blocks - 1) / blocks);
    const int c = (int)std::min<int64_t>(want, std::max(1, n_oth / least));
    *len = ceil_to(ceil_to(n_oth, c), unit) * unit;
    *chunks = ceil_to(n_oth, *len);
}

// Enough waves to fill 256 CUs: two workgroups of four waves per SIMD's share.
constexpr int kTargetBlocks = 2048;

Split owner_split(const DenseDev &D)
{
    Split s;
    s.blocks_r = ceil_to(D.N, kBlock);
    s.blocks_c = ceil_to(D.M, kBlock);
    chunk_up((int64_t)D.B * s.blocks_r, D.M, kTargetBlocks / 2, 64, 1, &s.chunks_r, &s.len_r);
    chunk_up((int64_t)D.B * s.blocks_c, D.N, kTargetBlocks / 2, 64, 1, &s.chunks_c, &s.len_c);
    return s;
}

// Partial sums per column, one per row block, that a sweep adds up itself
// (every block reads them all, from beyond its L2); more are added by a launch
// of its own (5 us).
constexpr int kOwnParts = 16;
constexpr int kMostParts = 128;
constexpr int kSweepMax = 8192; // longest rows of k_dsweep

int sweep_waves(int M) { return M <= 512 ? 1 : M <= 1024 ? 2 : M <= 2048 ? 4 : M <= 4096 ? 8 : 16; }

// Row blocks per sample and rows per block of the sweeps: 16 blocks where they
// hold 2048 waves (32 x 2048 x 2048: 103 us a sweep, against 117 with 32), else
// more, of at least 16 rows: with few waves on a SIMD the time is that of a
// block's chain of row groups, about a microsecond each (1 x 2048 x 2048:
// 25 us a sweep with 32 blocks, 15 with 128).
void row_blocks(const DenseDev &D, int *nb, int *rb)
{
    const int64_t waves = (int64_t)D.B * (D.M <= kSweepMax ? sweep_waves(D.M) : 16);
    const int n = std::max(1, std::min({kMostParts, std::max(kOwnParts, ceil_to(2048, waves)), D.N / 16}));
    *rb = ceil_to(ceil_to(D.N, n), 4) * 4;
    *nb = ceil_to(D.N, *rb);
}

// e_l of the stored scalings.
int drift(const DenseDev &D, int l)
{
    if (l >= D.L)
        l = D.L - 1;
    return l <= 0 ? 0 : (int)std::lrint(l * std::log2((double)D.N / D.M));
}
double pow2(int e) { return std::ldexp(1.0, e); }

template <DenseMode MODE> void launch_sweep(const DenseDev &D, const Sweep &s, int samples, hipStream_t st)
{
    const dim3 grid(samples * s.nb);
    if (D.M <= 256)
        hipLaunchKernelGGL((k_dsweep<MODE, 1, 1>), grid, dim3(64), 0, st, D, s);
    else
        switch (sweep_waves(D.M)) {
        case 1: hipLaunchKernelGGL((k_dsweep<MODE, 1, 2>), grid, dim3(64), 0, st, D, s); break;
        case 2: hipLaunchKernelGGL((k_dsweep<MODE, 2, 2>), grid, dim3(128), 0, st, D, s); break;
        case 4: hipLaunchKernelGGL((k_dsweep<MODE, 4, 2>), grid, dim3(256), 0, st, D, s); break;
        case 8: hipLaunchKernelGGL((k_dsweep<MODE, 8, 2>), grid, dim3(512), 0, st, D, s); break;
        default: hipLaunchKernelGGL((k_dsweep<MODE, 16, 2>), grid, dim3(1024), 0, st, D, s); break;
        }
}

// One iteration of all samples: the fused sweep, or, for rows too long for
// it, the column values, the row products and the column sums in turn.
template <DenseMode MODE> void iteration(const DenseDev &D, Sweep s, hipStream_t st)
{
    constexpr int OP = MODE == FWD ? ROW_FWD : ROW_BWD;
    const unsigned cols = blocks_for((int64_t)D.B * D.M, kBlock);
    if (D.M <= kSweepMax) {
        if (s.parts > kOwnParts) {
            hipLaunchKernelGGL(k_dcolumns<MODE>, dim3(cols), dim3(kBlock), 0, st, D, s);
            s.parts = 0;
        }
        launch_sweep<MODE>(D, s, D.B, st);
        return;
    }
    hipLaunchKernelGGL(k_dcolumns<MODE>, dim3(cols), dim3(kBlock), 0, st, D, s);
    const unsigned groups = blocks_for((int64_t)D.B * ceil_to(D.N, 4), kBlock / 64);
    hipLaunchKernelGGL((k_drow<OP, 2>), dim3(groups), dim3(kBlock), 0, st, D, s);
    if (s.part_out) {
        const double *w = MODE == FWD ? D.row.sc + (size_t)s.l * D.B * D.N : D.row.sb + (size_t)(s.l - 2) * D.B * D.N;
        hipLaunchKernelGGL((k_dcol<COL_W, 2>), dim3(D.B * s.nb * ceil_to(D.ld, kBlock)), dim3(kBlock), 0, st, D, s, w);
    }
}

template <int DP, bool ROWS, bool GRAD> void launch_pair(const DenseDev &D, hipStream_t st)
{
    const int n_own = ROWS ? D.N : D.M, n_oth = ROWS ? D.M : D.N, tiles = ceil_to(n_own, 64);
    int chunks, len;
    dense_pair_chunks(D.B, n_own, n_oth, &chunks, &len);
    hipLaunchKernelGGL((k_dpair<DP, ROWS, GRAD>), dim3(D.B * tiles * chunks), dim3(kBlock), 0, st, D, tiles, chunks, len,
                       D.pair);
    const unsigned owners = blocks_for((int64_t)D.B * n_own, kBlock);
    if (GRAD)
        hipLaunchKernelGGL(k_dgrad<DP>, dim3(owners), dim3(kBlock), 0, st, D, ROWS ? 1 : 0, chunks, (const double *)D.pair);
    else
        hipLaunchKernelGGL(k_dsigma, dim3(owners), dim3(kBlock), 0, st, D, ROWS ? 1 : 0, chunks, (const double *)D.pair);
}

template <int DP> void forward_dp(const DenseDev &D, double lk_row, double lk_col, hipStream_t st)
{
    const int64_t BN = (int64_t)D.B * D.N, BM = (int64_t)D.B * D.M;
    const Split sp = owner_split(D);
    const dim3 owners(blocks_for(BN + BM, kBlock)), block(kBlock);
    const dim3 both(D.B * (sp.blocks_r * sp.chunks_r + sp.blocks_c * sp.chunks_c));
    hipLaunchKernelGGL(k_dprep, dim3(blocks_for((BN + BM) * DP, kBlock)), block, 0, st, D);
    hipLaunchKernelGGL(k_dmin<DP>, both, block, 0, st, D, sp, (float4 *)D.owner_part);
    hipLaunchKernelGGL(k_dstat<DP>, owners, block, 0, st, D, sp, (const float4 *)D.owner_part, lk_row, lk_col);
    hipLaunchKernelGGL(k_dz<DP>, both, block, 0, st, D, sp, D.owner_part);
    hipLaunchKernelGGL(k_dzsum, owners, block, 0, st, D, sp, (const double *)D.owner_part);
    Sweep s{};
    row_blocks(D, &s.nb, &s.rb);
    const int cb = ceil_to(D.ld, kBlock);
    hipLaunchKernelGGL(k_dp0<DP>, dim3(D.B * s.nb * cb), block, 0, st, D, s.rb, s.nb, D.part[0]);
    for (int l = 1; l <= D.L; ++l) {
        s.l = l;
        s.parts = s.nb;
        s.part_in = D.part[(l - 1) & 1];
        s.part_out = l < D.L ? D.part[l & 1] : nullptr;
        s.f_in = pow2(drift(D, l - 1) - drift(D, l - 2));
        s.f_out = pow2(drift(D, l - 1) - drift(D, l));
        iteration<FWD>(D, s, st);
    }
    hipLaunchKernelGGL((k_drow<ROW_LOSS, DP>), dim3(blocks_for((int64_t)D.B * ceil_to(D.N, 4), kBlock / 64)), block, 0,
                       st, D, s);
    hipLaunchKernelGGL(k_dloss_sum, dim3(D.B), block, 0, st, D);
}

template <int DP> void backward_dp(const DenseDev &D, hipStream_t st)
{
    const dim3 block(kBlock);
    if (D.L > 0) {
        Sweep s{};
        row_blocks(D, &s.nb, &s.rb);
        hipLaunchKernelGGL(k_drbar, dim3(blocks_for((int64_t)D.B * D.N, kBlock)), block, 0, st, D);
        s.part_out = D.part[0];
        hipLaunchKernelGGL((k_dcol<COL_DIRECT, DP>), dim3(D.B * s.nb * ceil_to(D.ld, kBlock)), block, 0, st, D, s,
                           (const double *)(D.row.sb + (size_t)(D.L - 1) * D.B * D.N));
        int turn = 0;
        for (int l = D.L; l >= 1; --l, turn ^= 1) {
            s.l = l;
            s.parts = s.nb;
            s.part_in = D.part[turn];
            s.part_out = D.part[turn ^ 1];
            s.f_in = D.eps_stab * pow2(drift(D, l - 1) - drift(D, l));
            s.f_out = pow2(drift(D, l - 1) - drift(D, l - 2));
            if (l > 1)
                iteration<BWD>(D, s, st);
            else // Rbar^0 is not needed
                hipLaunchKernelGGL(k_dcolumns<BWD>, dim3(blocks_for((int64_t)D.B * D.M, kBlock)), block, 0, st, D, s);
        }
    }
    launch_pair<DP, true, false>(D, st);
    launch_pair<DP, false, false>(D, st);
    launch_pair<DP, true, true>(D, st);
    if (D.grad_y)
        launch_pair<DP, false, true>(D, st);
}

} // namespace

int dense_padded_dim(int d) { return d <= 2 ? 2 : d <= 4 ? d : d <= 8 ? 8 : 16; }

void dense_pair_chunks(int B, int n_own, int n_oth, int *chunks, int *len)
{
    chunk_up((int64_t)B * ceil_to(n_own, 64), n_oth, 1024, kPairT, kPairT, chunks, len);
}

DenseScratch dense_scratch(const DenseDev &D)
{
    const size_t BN = (size_t)D.B * D.N, BM = (size_t)D.B * D.M;
    const Split sp = owner_split(D);
    int nb, rb, cr, cc, len;
    row_blocks(D, &nb, &rb);
    dense_pair_chunks(D.B, D.N, D.M, &cr, &len);
    dense_pair_chunks(D.B, D.M, D.N, &cc, &len);
    DenseScratch s;
    s.owner = 2 * ((size_t)sp.chunks_r * BN + (size_t)sp.chunks_c * BM); // float4 of the minima; half for the sums
    s.part = (size_t)D.B * nb * D.ld;
    s.pair = std::max((size_t)cr * BN, (size_t)cc * BM) * std::max(3, D.dp);
    return s;
}

void launch_dense_forward(const DenseDev &D, double lk_row, double lk_col, hipStream_t s)
{
    switch (D.dp) {
    case 2: forward_dp<2>(D, lk_row, lk_col, s); break;
    case 3: forward_dp<3>(D, lk_row, lk_col, s); break;
    case 4: forward_dp<4>(D, lk_row, lk_col, s); break;
    case 8: forward_dp<8>(D, lk_row, lk_col, s); break;
    default: forward_dp<16>(D, lk_row, lk_col, s); break;
    }
}

void launch_dense_backward(const DenseDev &D, hipStream_t s)
{
    switch (D.dp) {
    case 2: backward_dp<2>(D, s); break;
    case 3: backward_dp<3>(D, s); break;
    case 4: backward_dp<4>(D, s); break;
    case 8: backward_dp<8>(D, s); break;
    default: backward_dp<16>(D, s); break;
    }
}

} // namespace apml
