// Sinkhorn normalisation on the stored pairs (Eq. 3, Eq. 4; Alg. 1 steps
// 4-7), the loss (Sec. III-D) and the reverse Sinkhorn sweeps.
//
// Scaling form. Every column step of Eq. 3 divides a whole column by one
// factor and every row step of Eq. 4 a whole row, so after iteration l the
// plan is v = alpha^l_i P0_ij beta^l_j with
//   beta^l_j  = beta^(l-1)_j  / (beta^(l-1)_j  sum_i alpha^(l-1)_i P0_ij + eps)
//   alpha^l_i = alpha^(l-1)_i / (alpha^(l-1)_i sum_j P0_ij beta^l_j     + eps)
// which is Eq. 3 / Eq. 4 exactly, including eps. A sweep reads P0 and the
// indices once and writes no per-pair values.
//
// Per-sample kernels: one 1024-lane workgroup per sample runs all 2L sweeps
// with the sample's pairs in registers. k_place and the column softmax cut every
// row's (column's) pairs into pieces of kP and lay them out so that an
// owner's pieces are consecutive lanes of one wave (see PackedOrder). In a
// sweep each lane sums its pieces (gathering the other side's values from
// LDS) and the pieces of one owner are added by a butterfly inside their
// aligned lane group, in a fixed order. In the forward kernel the group's
// first lane then applies its owner's scaling at once (one barrier per
// sweep); in the reverse kernel it applies its owner's recurrence.
// Sums have a fixed association, so results are bitwise reproducible.
//
// Reverse sweeps: the adjoints of the row and column sums of P0 against the
// scalings follow one another through two short recurrences (see the
// per-iteration reverse launches below), with no per-pair state but the sum of
// each pair's terms, which becomes dLoss/dP0.
#include <algorithm>
#include <atomic>
#include <cstdlib>

#include "apml_internal.h"
#include "device_common.h"
#include "pieces.h"

namespace apml {
namespace {

constexpr int kT = kSinkLanes;
constexpr int kP = kSinkPiece;
constexpr int kSL = kSinkOwners / kSinkLanes; // owners per lane in the owner phase
using pieces::pk_index;
using pieces::place_order;

__global__ __launch_bounds__(kT) void k_place(DevPlan d, int32_t *place)
{
    __shared__ int hist[8], base[8];
    place_order(d, place, blockIdx.x, blockIdx.y == 0, hist, base);
}

// ---------------------------------------------------------------------------
// per-sample kernels
// ---------------------------------------------------------------------------

// A lane's positions of one order, in registers for the whole kernel.
template <int SLP> struct Pieces {
    float p0[SLP][kP];
    uint32_t gi[SLP][kP / 2];
    uint32_t info[SLP];
    int n; // positions used (wave-uniform)
};

// The first SLP of the layout's slots.
template <int SLP> __device__ void load_pieces(Pieces<SLP> &pc, const PackedOrder &pk, int b)
{
    const int tid = threadIdx.x;
#pragma unroll
    for (int s = 0; s < SLP; ++s) {
        const int p = s * kT + tid;
#pragma unroll
        for (int e = 0; e < kP; ++e)
            pc.p0[s][e] = pk.p0[pk_index(b, p, e, kP, pk.slots)];
#pragma unroll
        for (int w = 0; w < kP / 2; ++w)
            pc.gi[s][w] = pk.gi[pk_index(b, p, w, kP / 2, pk.slots)];
        pc.info[s] = pk.info[pk_index(b, p, 0, 1, pk.slots)];
    }
    pc.n = __builtin_amdgcn_readfirstlane(pk.n_pos[b]);
}

// Unpacking of the cached words. Each 16-bit half of a gi word holds the byte
// offset of the gathered 8-byte value; an info word is owner (bits 0-10) | log2 group (11-13) | head (14)
// | valid (15) | first row-major position of a row piece (16-31). Bit fields
// are extracted at a base offset the compiler cannot see through (Unpack,
// renewed every sweep), so the unpacked values and the masks derived from
// them are recomputed inside the sweep loop instead of being hoisted out of
// it, which would multiply the registers held; P0 is widened to double by an
// instruction of its own for the same reason. The loads of a slot are issued
// before any of its arithmetic. Padding pairs carry P0 = 0 and offset 0:
// they gather real data and add nothing.
struct Unpack {
    uint32_t lo; // 0

    __device__ __forceinline__ static Unpack make()
    {
        Unpack u{0u};
        asm volatile("" : "+s"(u.lo));
        return u;
    }
    __device__ __forceinline__ uint32_t bits(uint32_t w, uint32_t pos, uint32_t width) const
    {
        return __builtin_amdgcn_ubfe(w, lo + pos, width);
    }
    __device__ __forceinline__ uint32_t half(uint32_t w, int e) const { return bits(w, (e & 1) ? 16u : 0u, 16u); }
    __device__ __forceinline__ int owner(uint32_t info) const { return (int)bits(info, 0, 11); }
    __device__ __forceinline__ int run(uint32_t info) const { return (int)bits(info, 16, 16); }
};

__device__ __forceinline__ double widen(float f)
{
    double d;
    asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(d) : "v"(f));
    return d;
}

template <typename T> __device__ __forceinline__ T lds_at(const void *base, uint32_t byte_off)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + byte_off);
}

// Slot s of this wave holds at least one used position.
__device__ __forceinline__ bool wave_active(int n_pos, int s)
{
    return s * kT + (int)(threadIdx.x & ~63u) < n_pos;
}

// Sum over the pairs of slot s of P0 times the gathered value (doubles at
// vals + byte offset), in pair order.
// P0 of slot s in double: widened once per kernel when the registers allow
// (WIDE), else widened at each use.
template <int SLP, bool WIDE> struct P0Cache {
    double v[WIDE ? SLP : 1][WIDE ? kP : 1];

    __device__ __forceinline__ void init(const Pieces<SLP> &pc)
    {
        if constexpr (WIDE) {
#pragma unroll
            for (int s = 0; s < SLP; ++s)
#pragma unroll
                for (int e = 0; e < kP; ++e)
                    v[s][e] = (double)pc.p0[s][e];
        }
    }
    __device__ __forceinline__ double get(const Pieces<SLP> &pc, int s, int e) const
    {
        if constexpr (WIDE)
            return v[s][e];
        else
            return widen(pc.p0[s][e]);
    }
};

template <int SLP, bool WIDE>
__device__ __forceinline__ double slot_dot(const Pieces<SLP> &pc, const P0Cache<SLP, WIDE> &p0, int s,
                                           const double *vals, const Unpack &u)
{
    double g[kP];
#pragma unroll
    for (int e = 0; e < kP; ++e)
        g[e] = lds_at<double>(vals, u.half(pc.gi[s][e / 2], e));
    double acc = p0.get(pc, s, 0) * g[0];
#pragma unroll
    for (int e = 1; e < kP; ++e)
        acc = __builtin_fma(p0.get(pc, s, e), g[e], acc);
    return acc;
}

template <int K> __device__ __forceinline__ void bfly_step(double &acc, int lg, int lgmax)
{
    if (K < lgmax) { // wave-uniform
        const double y = partner<K>(acc);
        if (K < lg)
            acc += y;
    }
}

// Adds the partial sums of each aligned group of 2^lg lanes (lg from info);
// every lane of a group ends with the same bits (each step adds two values
// that are the same on both sides, and addition commutes). Groups are sorted
// by size, so the wave's first lane has the largest.
__device__ __forceinline__ double group_reduce(double acc, uint32_t info, const Unpack &u)
{
    const int lg = (int)u.bits(info, 11, 3);
    const int lgmax = __builtin_amdgcn_readfirstlane(lg);
    bfly_step<0>(acc, lg, lgmax);
    bfly_step<1>(acc, lg, lgmax);
    bfly_step<2>(acc, lg, lgmax);
    bfly_step<3>(acc, lg, lgmax);
    bfly_step<4>(acc, lg, lgmax);
    bfly_step<5>(acc, lg, lgmax);
    return acc;
}

// a / b for positive normal a, b: the hardware reciprocal refined by two
// Newton steps, then one correction of the quotient (within an ulp of the
// correctly rounded quotient; no scaling for denormals or overflow).
__device__ __forceinline__ double quotient(double a, double b)
{
    double r = __builtin_amdgcn_rcp(b);
    r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
    const double q = a * r;
    return __builtin_fma(r, __builtin_fma(-b, q, a), q);
}

// Up to this many slots the forward kernel keeps P0 in double in registers.
constexpr int kFwdWideSlots = 4;

// The head lane of an owner's group applies the owner's scaling as soon as
// the group has its sum: v = cur / (cur * sum + eps) (Eq. 3 or Eq. 4), into
// the owner's side array in LDS (which the phase does not gather from) and
// into the saved scalings.
__device__ __forceinline__ void apply_scaling(double acc, uint32_t info, double *own, double eps, double *g_val,
                                              const Unpack &u)
{
    if (u.bits(info, 14, 2) == 3u) { // head and valid
        const int o = u.owner(info);
        const double cur = own[o];
        const double den = cur * acc + eps;
        const double v = quotient(cur, den);
        own[o] = v;
        g_val[o] = v;
    }
}

// loss = sum_t v_t C_t (Sec. III-D) of sample b, with v = alpha P0 beta from
// the final scalings va, vb in LDS, over the sample's pairs [lo, hi) in
// row-major order, four pairs per lane in flight; part: kT / 64 doubles of LDS.
__device__ void sample_loss(const DevPlan &d, int b, int lo, int hi, const double *va, const double *vb, double *part)
{
    const int tid = threadIdx.x, N = d.N;
    double acc = 0.0;
    for (int t0 = lo + tid; t0 < hi; t0 += 4 * kT) {
        int r[4], c[4];
        float p[4];
        double C[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = t0 + u * kT < hi ? t0 + u * kT : lo;
            r[u] = d.csr_row[t] - b * N;
            c[u] = d.csr_col[t];
            p[u] = d.p0r[t];
            C[u] = d.cost[t];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (t0 + u * kT < hi)
                acc += va[r[u]] * (double)p[u] * vb[c[u]] * C[u];
    }
    acc = wave_sum(acc);
    if (lane_id() == 0)
        part[tid >> 6] = acc;
    lds_barrier();
    if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < kT / 64; ++w)
            s += part[w];
        d.loss[b] = (float)s;
    }
}

template <int SLP> __global__ __launch_bounds__(kT) void k_sinkhorn_fwd(DevPlan d, double eps)
{
    // static arrays: their addresses are constants folded into the LDS instructions
    __shared__ double va[kSinkOwners], vb[kSinkOwners], part[kT / 64];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int N = d.N, M = d.M, L = d.L;
    const size_t BN = (size_t)d.B * N, BM = (size_t)d.B * M;
    const int lo = d.row_ptr[(size_t)b * N], hi = d.row_ptr[(size_t)(b + 1) * N];
    Pieces<SLP> pr, pc;
    load_pieces(pr, d.pk_row, b);
    load_pieces(pc, d.pk_col, b);
    constexpr bool kWide = SLP <= kFwdWideSlots;
    P0Cache<SLP, kWide> prw, pcw;
    prw.init(pr);
    pcw.init(pc);
#pragma unroll
    for (int s = 0; s < kSL; ++s) {
        const int k = kSL * tid + s;
        if (k < N) {
            va[k] = 1.0;
            d.alpha[(size_t)b * N + k] = 1.0;
        }
        if (k < M) {
            vb[k] = 1.0;
            d.beta[(size_t)b * M + k] = 1.0;
        }
    }
    lds_barrier();

    for (int l = 1; l <= L; ++l) {
        const Unpack u = Unpack::make();
        // column scaling (Eq. 3): beta_j /= beta_j sum_i alpha_i P0_ij + eps
        double *gb = d.beta + l * BM + (size_t)b * M;
#pragma unroll
        for (int s = 0; s < SLP; ++s)
            if (wave_active(pc.n, s)) {
                const double acc = slot_dot(pc, pcw, s, va, u);
                apply_scaling(group_reduce(acc, pc.info[s], u), pc.info[s], vb, eps, gb, u);
            }
        lds_barrier();
        // row scaling (Eq. 4): alpha_i /= alpha_i sum_j P0_ij beta_j + eps
        double *ga = d.alpha + l * BN + (size_t)b * N;
#pragma unroll
        for (int s = 0; s < SLP; ++s)
            if (wave_active(pr.n, s)) {
                const double acc = slot_dot(pr, prw, s, vb, u);
                apply_scaling(group_reduce(acc, pr.info[s], u), pr.info[s], va, eps, ga, u);
            }
        lds_barrier();
    }

    sample_loss(d, b, lo, hi, va, vb, part);
}

// A row piece that holds pairs: valid and either the row's first piece or one
// with a position (a padding piece of a group has neither; a later real
// piece starts at least kP pairs into its row).
__device__ __forceinline__ bool real_piece(uint32_t info, const Unpack &u)
{
    return (info & 0x8000u) != 0 && (u.bits(info, 14, 1) != 0 || u.run(info) != 0);
}

// One slot of column pieces, from registers or from LDS.
struct ColSlot {
    float p0[kP];
    uint32_t gi[kP / 2];
    uint32_t info;
};
constexpr int kColSlotWords = kP + kP / 2 + 1;

// Column slots the reverse kernel keeps in LDS (28 KB each): the row pieces
// and the pairs' sums in double fill the registers of a lane beyond four slots.
__host__ __device__ constexpr int bwd_lds_slots(int slots) { return slots <= 3 ? 0 : slots == 4 ? 1 : 2; }

// Reverse sweeps of a sample in one workgroup: the recurrences of the
// per-iteration reverse launches, the pairs' sums in registers in row order.
// Per iteration a column phase (gathers Rbar), a row phase (gathers beta and
// Sbar) and two barriers; the scalings of the next phase's owners are staged
// in LDS by the lanes, two owners each. 32 x 2048 points: 63 us, and 11 for
// k_bwd_direct, whose loads of costs and coordinates would take this launch's
// few CUs 15 us more; with the plan adjoint itself per pair in LDS, in single
// precision, and an owner phase after each piece phase 77 us (16 x 1024: 31
// and 5 against 42). Gradients against 64 bits: 1.6e-7 -> 4e-8, and 5.6e-6 ->
// 8e-8 where two nearest points are almost equidistant.
template <int SLP> __global__ __launch_bounds__(kT) void k_sinkhorn_bwd(DevPlan d, double eps)
{
    constexpr int LC = bwd_lds_slots(SLP), RC = SLP - LC;
    __shared__ double2 cs[kSinkOwners];                  // (beta^l_j, Sbar^l_j)
    __shared__ double rb[kSinkOwners];                   // Rbar^l_i
    __shared__ double own_a[kSinkOwners], own_b[kSinkOwners]; // the owners' scalings of the coming phase
    extern __shared__ uint32_t lds_col[];                // [LC][kColSlotWords][kT]
    const int b = blockIdx.x, tid = threadIdx.x;
    const int N = d.N, M = d.M, L = d.L;
    const size_t BN = (size_t)d.B * N, BM = (size_t)d.B * M;
    const int lo = d.row_ptr[(size_t)b * N];
    Pieces<SLP> pr;
    Pieces<RC> pc;
    load_pieces(pr, d.pk_row, b);
    load_pieces(pc, d.pk_col, b);
#pragma unroll
    for (int s = 0; s < LC; ++s) { // read back by the same lane only
        const int p = (RC + s) * kT + tid;
#pragma unroll
        for (int e = 0; e < kP; ++e)
            lds_col[(s * kColSlotWords + e) * kT + tid] =
                __builtin_bit_cast(uint32_t, d.pk_col.p0[pk_index(b, p, e, kP, SLP)]);
#pragma unroll
        for (int w = 0; w < kP / 2; ++w)
            lds_col[(s * kColSlotWords + kP + w) * kT + tid] = d.pk_col.gi[pk_index(b, p, w, kP / 2, SLP)];
        lds_col[(s * kColSlotWords + kP + kP / 2) * kT + tid] = d.pk_col.info[pk_index(b, p, 0, 1, SLP)];
    }
    auto col_slot = [&](int s) {
        ColSlot c;
        if (s < RC) {
#pragma unroll
            for (int e = 0; e < kP; ++e)
                c.p0[e] = pc.p0[s][e];
#pragma unroll
            for (int w = 0; w < kP / 2; ++w)
                c.gi[w] = pc.gi[s][w];
            c.info = pc.info[s];
        } else {
            const uint32_t *q = lds_col + (s - RC) * kColSlotWords * kT + tid;
#pragma unroll
            for (int e = 0; e < kP; ++e)
                c.p0[e] = __builtin_bit_cast(float, q[e * kT]);
#pragma unroll
            for (int w = 0; w < kP / 2; ++w)
                c.gi[w] = q[(kP + w) * kT];
            c.info = q[(kP + kP / 2) * kT];
        }
        return c;
    };
    const double *alpha = d.alpha + (size_t)b * N, *beta = d.beta + (size_t)b * M; // + l * BN, + l * BM
    // lane t stages the scalings of owners t and t + kT
    auto stage = [&](double *own, const double *g, int n) {
#pragma unroll
        for (int s = 0; s < kSL; ++s)
            if (s * kT + tid < n)
                own[s * kT + tid] = g[s * kT + tid];
    };
    stage(rb, d.rbar + (size_t)b * N, N);
    stage(own_b, beta + L * BM, M);
#pragma unroll
    for (int s = 0; s < kSL; ++s)
        if (s * kT + tid < M)
            cs[s * kT + tid].y = d.cs[(size_t)b * M + s * kT + tid].y;

    double z[SLP][kP];
#pragma unroll
    for (int s = 0; s < SLP; ++s)
#pragma unroll
        for (int e = 0; e < kP; ++e)
            z[s][e] = 0.0;
    lds_barrier();

    double keep = 1.0; // factor of the previous Sbar: 1 for the direct term, then eps
    for (int l = L; l >= 1; --l) {
        const Unpack u = Unpack::make();
        stage(own_a, alpha + (l - 1) * BN, N); // for the row phase
        // column phase: Sbar^l_j = eps Sbar^(l+1)_j - (beta^l_j)^2 sum_i P0_ij Rbar^l_i
#pragma unroll
        for (int s = 0; s < SLP; ++s)
            if (wave_active(pc.n, s)) {
                const ColSlot c = col_slot(s);
                double g[kP];
#pragma unroll
                for (int e = 0; e < kP; ++e)
                    g[e] = lds_at<double>(rb, u.half(c.gi[e / 2], e));
                double acc = widen(c.p0[0]) * g[0];
#pragma unroll
                for (int e = 1; e < kP; ++e)
                    acc = __builtin_fma(widen(c.p0[e]), g[e], acc);
                acc = group_reduce(acc, c.info, u);
                if (u.bits(c.info, 14, 2) == 3u) { // head and valid
                    const int j = u.owner(c.info);
                    const double bl = own_b[j];
                    cs[j] = make_double2(bl, keep * cs[j].y - bl * (bl * acc));
                }
            }
        keep = eps;
        lds_barrier();
        stage(own_b, beta + (l - 1) * BM, M); // for the next column phase
        // row phase: the pairs' terms of iteration l and
        // Rbar^(l-1)_i = eps Rbar^l_i - (alpha^(l-1)_i)^2 sum_j P0_ij Sbar^l_j
#pragma unroll
        for (int s = 0; s < SLP; ++s)
            if (wave_active(pr.n, s)) {
                const int i = u.owner(pr.info[s]);
                const double r = rb[i], al = own_a[i];
                double acc = 0.0;
#pragma unroll
                for (int h = 0; h < kP; h += 2) { // two gathers at a time: at five slots 16 bytes of scratch, at six 104; four spill more
                    const double2 g0 = lds_at<double2>(cs, 2 * u.half(pr.gi[s][h / 2], 0));
                    const double2 g1 = lds_at<double2>(cs, 2 * u.half(pr.gi[s][h / 2], 1));
                    z[s][h] = __builtin_fma(r, g0.x, __builtin_fma(al, g0.y, z[s][h]));
                    z[s][h + 1] = __builtin_fma(r, g1.x, __builtin_fma(al, g1.y, z[s][h + 1]));
                    const double p0 = widen(pr.p0[s][h]);
                    acc = h == 0 ? p0 * g0.y : __builtin_fma(p0, g0.y, acc);
                    acc = __builtin_fma(widen(pr.p0[s][h + 1]), g1.y, acc);
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc = group_reduce(acc, pr.info[s], u);
                if (u.bits(pr.info[s], 14, 2) == 3u)
                    rb[i] = eps * r - al * (al * acc);
            }
        lds_barrier();
    }
    // the pairs' sums in row-major order
    {
        const Unpack u = Unpack::make();
        int rend[SLP]; // end of each row piece's row, 0 for padding
#pragma unroll
        for (int s = 0; s < SLP; ++s)
            rend[s] = d.row_ptr[(size_t)b * N + u.owner(pr.info[s]) + 1] - lo;
#pragma unroll
        for (int s = 0; s < SLP; ++s)
            rend[s] = real_piece(pr.info[s], u) ? rend[s] : 0;
#pragma unroll
        for (int s = 0; s < SLP; ++s) {
            const int run = u.run(pr.info[s]);
#pragma unroll
            for (int e = 0; e < kP; ++e)
                if (run + e < rend[s])
                    d.adj[lo + run + e] = z[s][e];
        }
    }
}

// ---------------------------------------------------------------------------
// streamed per-sample kernels (samples of up to kSinkOwnersW points per side)
// ---------------------------------------------------------------------------
//
// One 1024-lane workgroup per sample runs all 2L sweeps, as above, but the
// pieces (too many for registers) are read from memory in every sweep, a slot
// at a time with the next slot's loads in flight. The forward kernel keeps
// both scaling vectors in LDS in double precision (2 x 64 KB); the reverse
// kernels (below, for one or several workgroups per sample) hold the vector
// that the phase gathers: Rbar, or beta and Sbar (128 KB).
constexpr int kSLW = kSinkOwnersW / kT; // owners per thread in the placement

// Placement of one order of sample b (grid B x 2): as place_order, for up to
// kSinkOwnersW owners and the wide info word. A wave ranks 64 owners that follow
// one another, so that among groups of one size neighbours in position are mostly
// neighbours in the sample: the sweeps' loads of the owners' saved scalings and
// words then meet in few cache lines. With eight owners a lane, one after another,
// every lane met a line of its own: 160 x 8192 points, 20 iterations, one workgroup
// a sample, reverse sweeps 2545 -> 1613 us, forward 875 -> 654; 64 x 3000, split,
// 127 -> 117 and 115 -> 100.
__global__ __launch_bounds__(kT) void k_place_w(DevPlan d, int32_t *place)
{
    __shared__ int hist[8], base[8];
    const int b = blockIdx.x, tid = threadIdx.x;
    const bool rows = blockIdx.y == 0;
    const int n_own = rows ? d.N : d.M;
    const int32_t *ptr = rows ? d.row_ptr + (size_t)b * d.N : d.col_ptr + (size_t)b * d.M;
    const WideOrder pk = rows ? d.wk_row : d.wk_col;
    const int slots = pk.slots, cap = slots * kT;
    {
        const size_t np0 = (size_t)slots * kP * kT, ngi = np0 / 2;
        for (size_t k = tid; k < np0; k += kT)
            pk.p0[(size_t)b * np0 + k] = 0.0f;
        for (size_t k = tid; k < ngi; k += kT)
            pk.gi[(size_t)b * ngi + k] = 0u;
    }
    if (tid < 8)
        hist[tid] = 0;
    __syncthreads();
    int lg[kSLW], rk[kSLW];
#pragma unroll
    for (int s = 0; s < kSLW; ++s) {
        const int k = s * kT + tid;
        lg[s] = -1;
        if (k < n_own) {
            lg[s] = sink_log2_group(sink_pieces(ptr[k + 1] - ptr[k]));
            rk[s] = atomicAdd(&hist[lg[s]], 1);
        }
    }
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int c = 6; c >= 0; --c) { // largest groups first: every group is aligned to its size
            base[c] = run;
            run += hist[c] << c;
        }
        base[7] = run;
        pk.n_pos[b] = run;
    }
    __syncthreads();
    for (int p = base[7] + tid; p < cap; p += kT) // unused positions: invalid
        pk.info[pk_index(b, p, 0, 1, slots)] = 0u;
#pragma unroll
    for (int s = 0; s < kSLW; ++s) {
        if (lg[s] < 0)
            continue;
        const int k = s * kT + tid, first = base[lg[s]] + (rk[s] << lg[s]);
        place[((size_t)b * 2 + (rows ? 0 : 1)) * kSinkOwnersW + k] = first;
        for (int q = 0; q < (1 << lg[s]); ++q)
            pk.info[pk_index(b, first + q, 0, 1, slots)] =
                (uint32_t)k | ((uint32_t)lg[s] << 13) | ((q == 0 ? 1u : 0u) << 16) | (1u << 17);
    }
}

// Writes every stored pair into its streamed piece, one thread per pair and order.
__global__ __launch_bounds__(kBlock) void k_pack_w(DevPlan d, const int32_t *place)
{
    const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool rows = g < d.nnz;
    const int64_t t = rows ? g : g - d.nnz;
    if (t >= d.nnz)
        return;
    int b, owner, off, other;
    float p0;
    if (rows) {
        const int r = d.csr_row[t];
        b = r / d.N;
        owner = r - b * d.N;
        off = (int)(t - d.row_ptr[r]);
        other = d.csr_col[t];
        p0 = d.p0r[t];
    } else {
        const int gc = d.csc_col[t];
        b = gc / d.M;
        owner = gc - b * d.M;
        off = (int)(t - d.col_ptr[gc]);
        other = d.csc_row[t];
        p0 = d.p0c[t];
    }
    const WideOrder &pk = rows ? d.wk_row : d.wk_col;
    const int p = place[((size_t)b * 2 + (rows ? 0 : 1)) * kSinkOwnersW + owner] + off / kP, e = off % kP;
    pk.p0[pk_index(b, p, e, kP, pk.slots)] = p0;
    reinterpret_cast<uint16_t *>(pk.gi + pk_index(b, p, e / 2, kP / 2, pk.slots))[e & 1] = (uint16_t)(other << 3);
}

// One streamed position of a lane: P0 of its pairs, the byte offsets of the
// gathered values, the info word.
struct WSlot {
    float p0[kP];
    uint32_t gi[kP / 2];
    uint32_t info;
};

template <class Order> __device__ __forceinline__ WSlot load_wslot(const Order &pk, int b, int s)
{
    WSlot w;
    const int p = s * kT + (int)threadIdx.x;
#pragma unroll
    for (int e = 0; e < kP; ++e)
        w.p0[e] = pk.p0[pk_index(b, p, e, kP, pk.slots)];
#pragma unroll
    for (int q = 0; q < kP / 2; ++q)
        w.gi[q] = pk.gi[pk_index(b, p, q, kP / 2, pk.slots)];
    w.info = pk.info[pk_index(b, p, 0, 1, pk.slots)];
    return w;
}

__device__ __forceinline__ double group_reduce_lg(double acc, int lg)
{
    const int lgmax = __builtin_amdgcn_readfirstlane(lg);
    bfly_step<0>(acc, lg, lgmax);
    bfly_step<1>(acc, lg, lgmax);
    bfly_step<2>(acc, lg, lgmax);
    bfly_step<3>(acc, lg, lgmax);
    bfly_step<4>(acc, lg, lgmax);
    bfly_step<5>(acc, lg, lgmax);
    return acc;
}

// Slots of the calling wave that hold used positions (wave-uniform).
__device__ __forceinline__ int wave_slots(int n_used)
{
    const int wave_base = (int)(threadIdx.x & ~63u);
    return wave_base < n_used ? (n_used - wave_base + kT - 1) / kT : 0;
}

// Slots whose loads are issued together before any of them is used: the
// streamed words come from the last-level cache, whose latency a single slot
// of work does not cover.
constexpr int kWBatch = 4;

// Split kernels: how a sample's workgroups exchange 64-bit words. When they
// all run on one XCD (local), through that XCD's L2: plain stores (the CU's
// cache writes through to the L2) and loads that skip only the CU's cache
// (sc0). Otherwise through memory: relaxed device-scope atomics, which skip
// the per-XCD L2s. Measured with 4 workgroups exchanging 8192 words: 2.3 us
// per meeting and exchange through the L2, 15.7 us through memory.
__device__ __forceinline__ void publish64(void *p, uint64_t v, bool local)
{
    if (local)
        *reinterpret_cast<uint64_t *>(p) = v;
    else
        __hip_atomic_store(reinterpret_cast<uint64_t *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One forward sweep: every owner's sum of P0 times the other side's scaling
// (vals) over its pieces, then its own scaling v = cur / (cur sum + eps)
// (Eq. 3 or Eq. 4) into own (LDS) and g_val (the saved scalings). With SPLIT
// the calling workgroup takes the slots s0, s0 + step, ... of each wave, and
// v goes to g_val only (published for the other workgroups of the sample);
// every owner's sum is formed by the same lanes as in the one-workgroup
// kernel, so both give the same bits.
template <bool SPLIT>
__device__ void wide_sweep(const WideOrder &pk, int b, int n_used, const double *vals, double *own, double eps,
                           double *g_val, int s0_first = 0, int step = 1, bool local = false)
{
    const int ns = wave_slots(n_used);
    for (int s0 = s0_first; s0 < ns; s0 += kWBatch * step) {
        WSlot w[kWBatch];
#pragma unroll
        for (int k = 0; k < kWBatch; ++k)
            if (s0 + k * step < ns)
                w[k] = load_wslot(pk, b, s0 + k * step);
#pragma unroll
        for (int k = 0; k < kWBatch; ++k) {
            if (s0 + k * step >= ns)
                break;
            const Unpack u = Unpack::make();
            double g[kP];
#pragma unroll
            for (int e = 0; e < kP; ++e)
                g[e] = lds_at<double>(vals, u.half(w[k].gi[e / 2], e));
            double acc = (double)w[k].p0[0] * g[0];
#pragma unroll
            for (int e = 1; e < kP; ++e)
                acc = __builtin_fma((double)w[k].p0[e], g[e], acc);
            acc = group_reduce_lg(acc, (int)u.bits(w[k].info, 13, 3));
            if (u.bits(w[k].info, 16, 2) == 3u) { // head and valid
                const int o = (int)u.bits(w[k].info, 0, 13);
                const double c = own[o];
                const double v = quotient(c, c * acc + eps);
                if constexpr (SPLIT) {
                    publish64(g_val + o, __builtin_bit_cast(uint64_t, v), local);
                } else {
                    own[o] = v;
                    g_val[o] = v;
                }
            }
        }
    }
}

__global__ __launch_bounds__(kT) void k_sinkhorn_fwd_w(DevPlan d, double eps)
{
    __shared__ double va[kSinkOwnersW], vb[kSinkOwnersW], part[kT / 64];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int N = d.N, M = d.M, L = d.L;
    const size_t BN = (size_t)d.B * N, BM = (size_t)d.B * M;
    const int lo = d.row_ptr[(size_t)b * N], hi = d.row_ptr[(size_t)(b + 1) * N];
    const int n_row = __builtin_amdgcn_readfirstlane(d.wk_row.n_pos[b]);
    const int n_col = __builtin_amdgcn_readfirstlane(d.wk_col.n_pos[b]);
    for (int k = tid; k < N; k += kT) {
        va[k] = 1.0;
        d.alpha[(size_t)b * N + k] = 1.0;
    }
    for (int k = tid; k < M; k += kT) {
        vb[k] = 1.0;
        d.beta[(size_t)b * M + k] = 1.0;
    }
    lds_barrier();
    for (int l = 1; l <= L; ++l) {
        // column scaling (Eq. 3), then row scaling (Eq. 4)
        wide_sweep<false>(d.wk_col, b, n_col, va, vb, eps, d.beta + l * BM + (size_t)b * M);
        lds_barrier();
        wide_sweep<false>(d.wk_row, b, n_row, vb, va, eps, d.alpha + l * BN + (size_t)b * N);
        lds_barrier();
    }
    sample_loss(d, b, lo, hi, va, vb, part);
}

// ---------------------------------------------------------------------------
// split streamed kernels: K workgroups per sample
// ---------------------------------------------------------------------------
//
// The streamed kernels above leave most CUs idle when the batch has fewer
// samples than the chip has CUs. Here K workgroups (one per CU) share a
// sample: workgroup k takes the slots k, k + K, ... of every wave, so each
// owner's sum is formed by the same lanes in the same order as in the
// one-workgroup kernels (same bits). After each half-sweep the owners' new
// values (the saved scalings, or the adjoints of the sums) are published to
// global memory and the K workgroups meet (split_meet), then every workgroup
// reads the whole vector into its LDS. The grid is launched cooperatively:
// all its workgroups are resident at once, so a meeting always completes.

constexpr unsigned kSplitSpinLimit = 1u << 20; // polls of one meeting (about a second) before giving up

// Sample and member of workgroup g, or false for a workgroup without one.
// Workgroups are dispatched to the eight XCDs in turn, so sample b takes
// XCD b % 8 and the ids x + 8 ((b / 8) K + k) on it: a sample's K workgroups
// share an XCD (their meetings stay within one L2's reach). The grid is
// split_grid(B, K) workgroups; those past the last sample end at once.
__device__ __forceinline__ bool split_member(int g, int B, int K, int &b, int &k)
{
    const int x = g % 8, slot = g / 8;
    b = (slot / K) * 8 + x;
    k = slot % K;
    return b < B;
}

// Meeting t of a sample's K workgroups (t = 1, 2, ...): each waits until its
// own stores have completed (s_waitcnt: plain stores have then reached the
// L2, device-scope atomic stores the level every XCD reads), counts itself
// in at the sample's counter, does the work of `shadow` and waits until all K
// have (target K t). The counter is a relaxed device-scope atomic, so no
// cache is written back or invalidated. The wait is bounded: past
// kSplitSpinLimit polls, or once another workgroup has given up, it sets bit
// 2 of the error word and returns false, and the caller ends. target 0: a
// sample of one workgroup, which only waits for itself.
template <class Shadow>
__device__ __forceinline__ bool split_meet(uint32_t *cnt, uint32_t target, unsigned int *err, int *stop, Shadow shadow)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (target != 0 && threadIdx.x == 0)
        __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    shadow();
    if (target != 0 && threadIdx.x == 0) {
        unsigned spins = 0;
        while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++spins > kSplitSpinLimit ||
                ((spins & 63u) == 0 && (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 4u))) {
                __hip_atomic_fetch_or(err, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *stop = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    __syncthreads();
    return *stop == 0;
}

__device__ __forceinline__ bool split_meet(uint32_t *cnt, uint32_t target, unsigned int *err, int *stop)
{
    return split_meet(cnt, target, err, stop, [] {});
}

// First meeting of a sample's workgroups: each records its XCD (hardware
// register XCC_ID) next to the counter, and all decide alike, from the same
// K words, whether they share one (local exchange through its L2).
__device__ bool split_begin(uint32_t *sync, int K, int k, unsigned int *err, int *stop, int *local)
{
    if (threadIdx.x == 0) {
        unsigned id;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(id));
        __hip_atomic_store(sync + 1 + k, id + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!split_meet(sync, (uint32_t)K, err, stop))
        return false;
    if (threadIdx.x == 0) {
        const unsigned first = __hip_atomic_load(sync + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int same = 1;
        for (int q = 1; q < K; ++q)
            same &= __hip_atomic_load(sync + 1 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == first;
        *local = same;
    }
    __syncthreads();
    return true;
}

// Eight published words per lane, word u of lane t at word u * lanes + t
// of the sample's vector, and the wait for them, in one asm statement, so
// that no use of a result can be placed before the wait.
//  local: through the L2 only (sc0: the loads skip the CU's cache); each
//  lane's offsets clamped to the vector's last word, so that no line outside
//  the vector is brought into the CU's cache (see split_gather).
//  else: from memory past the L2s (sc1, as relaxed device-scope atomic
//  loads), one offset register and a scalar base per chunk of lanes; the
//  caller's array extends 8 * lanes words past the vector's start.
#define APML_LDL(I, J) "global_load_dwordx2 %" #I ", %" #J ", %[base] sc0\n\t"
#define APML_LDM(I, B) "global_load_dwordx2 %" #I ", %[off], %" #B " sc1\n\t"
#define APML_OUT8                                                                                             \
    "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])

// The lane's index in the workgroup, opaque to the compiler: what is derived
// from it in a sweep's exchange (offsets, bounds, addresses of eight words) is
// formed there again instead of being held in registers across the sweeps.
__device__ __forceinline__ int fresh_lane()
{
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The sample's n published doubles (n <= 8 * lanes), each given to put (an LDS store).
template <class Put> __device__ __forceinline__ void split_gather(const double *g, int n, bool local, Put put)
{
    static_assert(kSinkOwnersW / kT == 8, "eight words per lane");
    // the base in scalar registers: each 32-bit half read from the first lane
    // (the builtin takes 32-bit values; a 64-bit argument would be cut)
    const int lane = fresh_lane();
    const uint64_t a = (uint64_t)(uintptr_t)g;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const uint64_t base = ((uint64_t)hi << 32) | lo;
    uint64_t v[8];
    if (local) {
        uint32_t off[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            off[u] = (uint32_t)min(u * kT + lane, n - 1) * 8u;
        asm volatile("buffer_inv sc0\n\t" // no line of an earlier read may serve these loads
                     APML_LDL(0, 8) APML_LDL(1, 9) APML_LDL(2, 10) APML_LDL(3, 11) APML_LDL(4, 12) APML_LDL(5, 13)
                     APML_LDL(6, 14) APML_LDL(7, 15) "s_waitcnt vmcnt(0)"
                     : APML_OUT8
                     : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "v"(off[4]), "v"(off[5]), "v"(off[6]),
                       "v"(off[7]), [base] "s"(reinterpret_cast<const void *>((uintptr_t)base))
                     : "memory");
    } else {
        const void *bs[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            bs[u] = reinterpret_cast<const void *>((uintptr_t)(base + (uint64_t)u * kT * 8u));
        const uint32_t off = (uint32_t)lane * 8u;
        asm volatile(APML_LDM(0, 8) APML_LDM(1, 9) APML_LDM(2, 10) APML_LDM(3, 11) APML_LDM(4, 12)
                         APML_LDM(5, 13) APML_LDM(6, 14) APML_LDM(7, 15) "s_waitcnt vmcnt(0)"
                     : APML_OUT8
                     : "s"(bs[0]), "s"(bs[1]), "s"(bs[2]), "s"(bs[3]), "s"(bs[4]), "s"(bs[5]), "s"(bs[6]),
                       "s"(bs[7]), [off] "v"(off)
                     : "memory");
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int o = u * kT + lane;
        if (o < n)
            put(o, __builtin_bit_cast(double, v[u]));
    }
}
#undef APML_OUT8
#undef APML_LDM
#undef APML_LDL

__global__ __launch_bounds__(kT) void k_sinkhorn_fwd_ws(DevPlan d, double eps, int K)
{
    __shared__ double va[kSinkOwnersW], vb[kSinkOwnersW], part[kT / 64];
    __shared__ int stop, local;
    int b, k;
    if (!split_member(blockIdx.x, d.B, K, b, k))
        return;
    const int tid = threadIdx.x;
    const int N = d.N, M = d.M, L = d.L;
    const size_t BN = (size_t)d.B * N, BM = (size_t)d.B * M;
    uint32_t *cnt = d.split_sync + ((size_t)b * 2 + 0) * kSplitSyncStride;
    const int n_row = __builtin_amdgcn_readfirstlane(d.wk_row.n_pos[b]);
    const int n_col = __builtin_amdgcn_readfirstlane(d.wk_col.n_pos[b]);
    for (int o = tid; o < N; o += kT) {
        va[o] = 1.0;
        if (k == 0)
            d.alpha[(size_t)b * N + o] = 1.0;
    }
    for (int o = tid; o < M; o += kT) {
        vb[o] = 1.0;
        if (k == 0)
            d.beta[(size_t)b * M + o] = 1.0;
    }
    if (tid == 0)
        stop = 0;
    lds_barrier();
    if (!split_begin(cnt, K, k, &d.ctr->error, &stop, &local))
        return;
    const bool loc = local != 0;
    uint32_t t = 1;
    for (int l = 1; l <= L; ++l) {
        // column scaling (Eq. 3) of this workgroup's owners, then all of them
        double *gb = d.beta + l * BM + (size_t)b * M;
        wide_sweep<true>(d.wk_col, b, n_col, va, vb, eps, gb, k, K, loc);
        if (!split_meet(cnt, (uint32_t)K * ++t, &d.ctr->error, &stop))
            return;
        split_gather(gb, M, loc, [&](int o, double v) { vb[o] = v; });
        lds_barrier();
        // row scaling (Eq. 4)
        double *ga = d.alpha + l * BN + (size_t)b * N;
        wide_sweep<true>(d.wk_row, b, n_row, vb, va, eps, ga, k, K, loc);
        if (!split_meet(cnt, (uint32_t)K * ++t, &d.ctr->error, &stop))
            return;
        split_gather(ga, N, loc, [&](int o, double v) { va[o] = v; });
        lds_barrier();
    }
    if (k == 0) // as the one-workgroup kernel, for the same bits
        sample_loss(d, b, d.row_ptr[(size_t)b * N], d.row_ptr[(size_t)(b + 1) * N], va, vb, part);
}

// The reverse sweeps (the recurrences of the per-iteration reverse launches)
// split over K workgroups, or in one (K = 1). After each phase the owners'
// heads publish their words, Sbar^l_j or Rbar^(l-1)_i, into a region of fresh
// memory for that phase (d.yc, d.yr: a word is never written twice within the
// kernel, so the exchange may go through the L2, as in the forward kernels);
// beta, the other factor of a row phase's gather, was saved by the forward
// kernel and is loaded in the meeting's shadow. Each pair's sum of terms is
// kept in double, streamed in the row pieces' layout (d.wz) or in registers.
// Keeping the adjoint itself per pair in both orders, in single precision, took
// twice the registers (three slots a lane at most, against four) or memory
// traffic: 64 x 8192 points, 20 iterations, step 1.95 -> 1.71 ms; gradients
// against 64 bits 1.3e-6 -> 5e-8.

// Words of one phase's region: whole cache lines, so that no line holds words of two phases.
__host__ __device__ inline size_t phase_region(size_t owners) { return (owners + 31) / 16 * 16; }

// The vectors of one sample in the reverse kernels.
struct RevSample {
    const double *alpha, *beta; // + l * BN, + l * BM
    const double *rbar;         // first Rbar
    const double2 *cs;          // first Sbar (.y)
    double *yr, *yc;            // regions: + (L - l) * sn, + (L - l) * sm
    size_t BN, BM, sn, sm;
};

__device__ __forceinline__ RevSample rev_sample(const DevPlan &d, int b)
{
    RevSample r;
    r.BN = (size_t)d.B * d.N;
    r.BM = (size_t)d.B * d.M;
    r.sn = phase_region(r.BN);
    r.sm = phase_region(r.BM);
    const size_t on = (size_t)b * d.N, om = (size_t)b * d.M;
    r.alpha = d.alpha + on;
    r.beta = d.beta + om;
    r.rbar = d.rbar + on;
    r.cs = d.cs + om;
    r.yr = d.yr + on;
    r.yc = d.yc + om;
    return r;
}

// The previous value of an owner's recurrence: the first one, or the word its head published last.
__device__ __forceinline__ double prev_s(const RevSample &r, int L, int l, int o)
{
    return l == L ? r.cs[o].y : r.yc[(size_t)(L - l - 1) * r.sm + o];
}
__device__ __forceinline__ double prev_r(const RevSample &r, int L, int l, int o)
{
    return l == L ? r.rbar[o] : r.yr[(size_t)(L - l - 1) * r.sn + o];
}

// Column phase of one slot: sum_i P0_ij Rbar_i over the pieces of an owner,
// and its new Sbar = keep old - beta^2 sum, published by the head.
__device__ __forceinline__ void rev_col_slot(const WSlot &w, const double *rb, double bl, double old, double *out,
                                             bool local)
{
    const Unpack u = Unpack::make();
    double g[kP];
#pragma unroll
    for (int e = 0; e < kP; ++e)
        g[e] = lds_at<double>(rb, u.half(w.gi[e / 2], e));
    double acc = widen(w.p0[0]) * g[0];
#pragma unroll
    for (int e = 1; e < kP; ++e)
        acc = __builtin_fma(widen(w.p0[e]), g[e], acc);
    acc = group_reduce_lg(acc, (int)u.bits(w.info, 13, 3));
    if (u.bits(w.info, 16, 2) == 3u) // head and valid
        publish64(out + u.bits(w.info, 0, 13), __builtin_bit_cast(uint64_t, old - bl * (bl * acc)), local);
}

// Row phase of one slot: the pairs' terms, the row's new Rbar = eps r - al^2
// sum_j P0_ij Sbar_j (the same in all lanes of the group), published by the head.
__device__ __forceinline__ double rev_row_slot(const WSlot &w, const double2 *cs, double r, double al, double eps,
                                               double (&z)[kP], double *out, bool local)
{
    const Unpack u = Unpack::make();
    double acc = 0.0;
#pragma unroll
    for (int h = 0; h < kP; h += 2) { // two gathers at a time keep the registers down
        const double2 g0 = lds_at<double2>(cs, 2 * u.half(w.gi[h / 2], 0));
        const double2 g1 = lds_at<double2>(cs, 2 * u.half(w.gi[h / 2], 1));
        z[h] = __builtin_fma(r, g0.x, __builtin_fma(al, g0.y, z[h]));
        z[h + 1] = __builtin_fma(r, g1.x, __builtin_fma(al, g1.y, z[h + 1]));
        acc = h == 0 ? widen(w.p0[h]) * g0.y : __builtin_fma(widen(w.p0[h]), g0.y, acc);
        acc = __builtin_fma(widen(w.p0[h + 1]), g1.y, acc);
        __builtin_amdgcn_sched_barrier(0);
    }
    acc = group_reduce_lg(acc, (int)u.bits(w.info, 13, 3));
    const double next = eps * r - al * (al * acc);
    if (u.bits(w.info, 16, 2) == 3u)
        publish64(out + u.bits(w.info, 0, 13), __builtin_bit_cast(uint64_t, next), local);
    return next;
}

// The sums of a slot's pairs into adj, row-major. p: the lane's position.
__device__ __forceinline__ void store_adj(const DevPlan &d, int b, const WSlot &w, int p, const double (&z)[kP])
{
    if ((w.info >> 17 & 1u) == 0u) // not a used position
        return;
    const int i = (int)(w.info & 0x1FFFu), lg = (int)(w.info >> 13 & 7u);
    const int q = p & ((1 << lg) - 1); // groups are aligned to their size
    const int r0 = d.row_ptr[(size_t)b * d.N + i], len = d.row_ptr[(size_t)b * d.N + i + 1] - r0;
#pragma unroll
    for (int e = 0; e < kP; ++e)
        if (q * kP + e < len)
            d.adj[r0 + q * kP + e] = z[e];
}

// The sweeps of a sample: cols(l, out, keep) and rows(l, out) form the owners'
// new words of a phase from the vector in buf and publish them; between the
// phases the workgroups meet and every one reads the whole vector.
template <class Cols, class Rows>
__device__ __forceinline__ void rev_sweeps(const DevPlan &d, double eps, int b, int k, int K, double2 *buf, int *stop,
                                           int *local, Cols cols, Rows rows)
{
    const int tid = threadIdx.x, N = d.N, M = d.M, L = d.L;
    const RevSample r = rev_sample(d, b);
    uint32_t *cnt = d.split_sync + ((size_t)b * 2 + 1) * kSplitSyncStride;
    double *rb = reinterpret_cast<double *>(buf);
    for (int o = tid; o < N; o += kT)
        rb[o] = r.rbar[o];
    if (tid == 0) {
        *stop = 0;
        *local = 1;
    }
    lds_barrier();
    if (K > 1 && !split_begin(cnt, K, k, &d.ctr->error, stop, local))
        return;
    const bool loc = *local != 0;
    uint32_t t = K > 1 ? 1 : 0;
    auto next = [&]() { return K > 1 ? (uint32_t)K * ++t : 0u; };
    double keep = 1.0; // factor of the previous Sbar: 1 for the direct term, then eps
    for (int l = L; l >= 1; --l) {
        double *yc = r.yc + (size_t)(L - l) * r.sm, *yr = r.yr + (size_t)(L - l) * r.sn;
        cols(r, l, keep, rb, yc, loc);
        keep = eps;
        const bool met = split_meet(cnt, next(), &d.ctr->error, stop, [&] {
            const double *beta = r.beta + (size_t)l * r.BM;
            const int lane = fresh_lane();
#pragma unroll
            for (int u = 0; u < kSinkOwnersW / kT; ++u)
                if (u * kT + lane < M)
                    buf[u * kT + lane].x = beta[u * kT + lane];
        });
        if (!met)
            return;
        split_gather(yc, M, loc, [&](int o, double v) { buf[o].y = v; });
        lds_barrier();
        rows(r, l, buf, yr, loc);
        if (l == 1)
            break;
        if (!split_meet(cnt, next(), &d.ctr->error, stop))
            return;
        split_gather(yr, N, loc, [&](int o, double v) { rb[o] = v; });
        lds_barrier();
    }
}

__global__ __launch_bounds__(kT) void k_sinkhorn_bwd_ws(DevPlan d, double eps, int K)
{
    __shared__ double2 buf[kSinkOwnersW];
    __shared__ int stop, local;
    int b, k;
    if (!split_member(blockIdx.x, d.B, K, b, k))
        return;
    const int tid = threadIdx.x, L = d.L;
    const int nr = wave_slots(__builtin_amdgcn_readfirstlane(d.wk_row.n_pos[b]));
    const int nc = wave_slots(__builtin_amdgcn_readfirstlane(d.wk_col.n_pos[b]));
    rev_sweeps(
        d, eps, b, k, K, buf, &stop, &local,
        [&](const RevSample &r, int l, double keep, const double *rb, double *yc, bool loc) {
            for (int s0 = k; s0 < nc; s0 += kWBatch * K) {
                WSlot w[kWBatch];
                double bl[kWBatch], old[kWBatch];
#pragma unroll
                for (int q = 0; q < kWBatch; ++q)
                    if (s0 + q * K < nc)
                        w[q] = load_wslot(d.wk_col, b, s0 + q * K);
#pragma unroll
                for (int q = 0; q < kWBatch; ++q)
                    if (s0 + q * K < nc) {
                        const int o = (int)(w[q].info & 0x1FFFu);
                        bl[q] = r.beta[(size_t)l * r.BM + o];
                        old[q] = keep * prev_s(r, L, l, o);
                    }
#pragma unroll
                for (int q = 0; q < kWBatch; ++q)
                    if (s0 + q * K < nc)
                        rev_col_slot(w[q], rb, bl[q], old[q], yc, loc);
            }
        },
        [&](const RevSample &r, int l, const double2 *cs, double *yr, bool loc) {
            for (int s0 = k; s0 < nr; s0 += kWBatch * K) {
                WSlot w[kWBatch];
                double al[kWBatch], old[kWBatch], z[kWBatch][kP];
#pragma unroll
                for (int q = 0; q < kWBatch; ++q)
                    if (s0 + q * K < nr) {
                        w[q] = load_wslot(d.wk_row, b, s0 + q * K);
                        const int p = (s0 + q * K) * kT + tid;
#pragma unroll
                        for (int e = 0; e < kP; ++e)
                            z[q][e] = l == L ? 0.0 : d.wz[pk_index(b, p, e, kP, d.wk_row.slots)];
                    }
#pragma unroll
                for (int q = 0; q < kWBatch; ++q)
                    if (s0 + q * K < nr) {
                        const int o = (int)(w[q].info & 0x1FFFu);
                        al[q] = r.alpha[(size_t)(l - 1) * r.BN + o];
                        old[q] = prev_r(r, L, l, o);
                    }
#pragma unroll
                for (int q = 0; q < kWBatch; ++q)
                    if (s0 + q * K < nr) {
                        rev_row_slot(w[q], cs, old[q], al[q], eps, z[q], yr, loc);
                        const int p = (s0 + q * K) * kT + tid;
                        if (l > 1) {
#pragma unroll
                            for (int e = 0; e < kP; ++e)
                                d.wz[pk_index(b, p, e, kP, d.wk_row.slots)] = z[q][e];
                        } else {
                            store_adj(d, b, w[q], p, z[q]);
                        }
                    }
            }
        });
}

// Register-resident split kernels: when a workgroup's share is at most SW
// slots per lane and order, its pieces (and in the reverse kernel its pairs'
// sums) are loaded once and kept in registers for every sweep, so a
// half-sweep reads nothing from memory but the owners' saved scalings and the
// exchanged vector. Same lanes, same arithmetic in the same order as the
// streamed kernels: the same bits.
constexpr int kSplitRegFwd = 3; // slots per lane and order held by the forward kernel
constexpr int kSplitRegBwd = 4; // and by the reverse kernel

// Slots of the calling wave that workgroup k of K takes (wave-uniform).
__device__ __forceinline__ int split_slots(int n_used, int k, int K)
{
    const int ns = wave_slots(n_used);
    return ns > k ? (ns - k + K - 1) / K : 0;
}

template <int SW, class Order>
__device__ __forceinline__ void load_my_slots(WSlot (&w)[SW], const Order &pk, int b, int n, int k, int K)
{
#pragma unroll
    for (int q = 0; q < SW; ++q)
        if (q < n)
            w[q] = load_wslot(pk, b, k + q * K);
}

// One forward half-sweep over the slots held in registers (as wide_sweep).
template <int SW>
__device__ __forceinline__ void reg_sweep(const WSlot (&w)[SW], int n, const double *vals, const double *own, double eps,
                                          double *g_val, bool local)
{
#pragma unroll
    for (int q = 0; q < SW; ++q) {
        if (q >= n)
            break;
        const Unpack u = Unpack::make();
        double g[kP];
#pragma unroll
        for (int e = 0; e < kP; ++e)
            g[e] = lds_at<double>(vals, u.half(w[q].gi[e / 2], e));
        double acc = (double)w[q].p0[0] * g[0];
#pragma unroll
        for (int e = 1; e < kP; ++e)
            acc = __builtin_fma((double)w[q].p0[e], g[e], acc);
        acc = group_reduce_lg(acc, (int)u.bits(w[q].info, 13, 3));
        if (u.bits(w[q].info, 16, 2) == 3u) { // head and valid
            const int o = (int)u.bits(w[q].info, 0, 13);
            const double c = own[o];
            publish64(g_val + o, __builtin_bit_cast(uint64_t, quotient(c, c * acc + eps)), local);
        }
    }
}

template <int SW> __global__ __launch_bounds__(kT) void k_sinkhorn_fwd_wr(DevPlan d, double eps, int K)
{
    __shared__ double va[kSinkOwnersW], vb[kSinkOwnersW], part[kT / 64];
    __shared__ int stop, local;
    int b, k;
    if (!split_member(blockIdx.x, d.B, K, b, k))
        return;
    const int tid = threadIdx.x;
    const int N = d.N, M = d.M, L = d.L;
    const size_t BN = (size_t)d.B * N, BM = (size_t)d.B * M;
    uint32_t *cnt = d.split_sync + ((size_t)b * 2 + 0) * kSplitSyncStride;
    const int mr = split_slots(__builtin_amdgcn_readfirstlane(d.wk_row.n_pos[b]), k, K);
    const int mc = split_slots(__builtin_amdgcn_readfirstlane(d.wk_col.n_pos[b]), k, K);
    WSlot pr[SW], pc[SW];
    load_my_slots(pr, d.wk_row, b, mr, k, K);
    load_my_slots(pc, d.wk_col, b, mc, k, K);
    for (int o = tid; o < N; o += kT) {
        va[o] = 1.0;
        if (k == 0)
            d.alpha[(size_t)b * N + o] = 1.0;
    }
    for (int o = tid; o < M; o += kT) {
        vb[o] = 1.0;
        if (k == 0)
            d.beta[(size_t)b * M + o] = 1.0;
    }
    if (tid == 0)
        stop = 0;
    lds_barrier();
    if (!split_begin(cnt, K, k, &d.ctr->error, &stop, &local))
        return;
    const bool loc = local != 0;
    uint32_t t = 1;
    for (int l = 1; l <= L; ++l) {
        double *gb = d.beta + l * BM + (size_t)b * M;
        reg_sweep(pc, mc, va, vb, eps, gb, loc); // Eq. 3
        if (!split_meet(cnt, (uint32_t)K * ++t, &d.ctr->error, &stop))
            return;
        split_gather(gb, M, loc, [&](int o, double v) { vb[o] = v; });
        lds_barrier();
        double *ga = d.alpha + l * BN + (size_t)b * N;
        reg_sweep(pr, mr, vb, va, eps, ga, loc); // Eq. 4
        if (!split_meet(cnt, (uint32_t)K * ++t, &d.ctr->error, &stop))
            return;
        split_gather(ga, N, loc, [&](int o, double v) { va[o] = v; });
        lds_barrier();
    }
    if (k == 0)
        sample_loss(d, b, d.row_ptr[(size_t)b * N], d.row_ptr[(size_t)(b + 1) * N], va, vb, part);
}

// The last of four column slots lives in LDS (28 KB beside the 128 KB of the
// gathered vector): with it too in registers, more than the 48 bytes of scratch that
// four slots take would spill.
__host__ __device__ constexpr int bwd_wide_lds_slots(int sw) { return sw == 4 ? 1 : 0; }

template <int SW> __global__ __launch_bounds__(kT) void k_sinkhorn_bwd_wr(DevPlan d, double eps, int K)
{
    constexpr int RC = SW - bwd_wide_lds_slots(SW);
    __shared__ double2 buf[kSinkOwnersW];
    __shared__ int stop, local;
    extern __shared__ uint32_t lds_col[]; // [SW - RC][kColSlotWords][kT]
    int b, k;
    if (!split_member(blockIdx.x, d.B, K, b, k))
        return;
    const int tid = threadIdx.x, L = d.L;
    const int mr = split_slots(__builtin_amdgcn_readfirstlane(d.wk_row.n_pos[b]), k, K);
    const int mc = split_slots(__builtin_amdgcn_readfirstlane(d.wk_col.n_pos[b]), k, K);
    WSlot pr[SW], pc[RC];
    load_my_slots(pr, d.wk_row, b, mr, k, K);
    load_my_slots(pc, d.wk_col, b, mc, k, K);
    if constexpr (SW > RC) { // read back by the same lane only
        if (RC < mc) {
            const WSlot w = load_wslot(d.wk_col, b, k + RC * K);
#pragma unroll
            for (int e = 0; e < kP; ++e)
                lds_col[e * kT + tid] = __builtin_bit_cast(uint32_t, w.p0[e]);
#pragma unroll
            for (int q = 0; q < kP / 2; ++q)
                lds_col[(kP + q) * kT + tid] = w.gi[q];
            lds_col[(kP + kP / 2) * kT + tid] = w.info;
        }
    }
    double z[SW][kP], old_r[SW];
#pragma unroll
    for (int q = 0; q < SW; ++q) {
        old_r[q] = 0.0;
#pragma unroll
        for (int e = 0; e < kP; ++e)
            z[q][e] = 0.0;
        if (q < mr)
            old_r[q] = d.rbar[(size_t)b * d.N + (pr[q].info & 0x1FFFu)];
    }
    rev_sweeps(
        d, eps, b, k, K, buf, &stop, &local,
        [&](const RevSample &r, int l, double keep, const double *rb, double *yc, bool loc) {
            double bl[SW], old[SW];
#pragma unroll
            for (int q = 0; q < SW; ++q)
                if (q < mc) {
                    const uint32_t info = q < RC ? pc[q < RC ? q : 0].info : lds_col[(kP + kP / 2) * kT + tid];
                    const int o = (int)Unpack::make().bits(info, 0, 13);
                    bl[q] = r.beta[(size_t)l * r.BM + o];
                    old[q] = keep * prev_s(r, L, l, o);
                }
#pragma unroll
            for (int q = 0; q < SW; ++q) {
                if (q >= mc)
                    break;
                if (q < RC) {
                    rev_col_slot(pc[q < RC ? q : 0], rb, bl[q], old[q], yc, loc);
                } else {
                    WSlot w;
#pragma unroll
                    for (int e = 0; e < kP; ++e)
                        w.p0[e] = __builtin_bit_cast(float, lds_col[e * kT + tid]);
#pragma unroll
                    for (int h = 0; h < kP / 2; ++h)
                        w.gi[h] = lds_col[(kP + h) * kT + tid];
                    w.info = lds_col[(kP + kP / 2) * kT + tid];
                    rev_col_slot(w, rb, bl[q], old[q], yc, loc);
                }
            }
        },
        [&](const RevSample &r, int l, const double2 *cs, double *yr, bool loc) {
            double al[SW];
#pragma unroll
            for (int q = 0; q < SW; ++q)
                if (q < mr)
                    al[q] = r.alpha[(size_t)(l - 1) * r.BN + Unpack::make().bits(pr[q].info, 0, 13)];
#pragma unroll
            for (int q = 0; q < SW; ++q) {
                if (q >= mr)
                    break;
                old_r[q] = rev_row_slot(pr[q], cs, old_r[q], al[q], eps, z[q], yr, loc);
                if (l == 1)
                    store_adj(d, b, pr[q], (k + q * K) * kT + tid, z[q]);
            }
        });
}

__global__ __launch_bounds__(kBlock) void k_zero_u32(uint32_t *a, int n)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k < n)
        a[k] = 0u;
}

// per-iteration kernels (any N, M): one launch per sweep
// ---------------------------------------------------------------------------
//
// G lanes per owner (row or column; steps_lanes), the whole wave for owners
// of more than G kSB pairs (each_owner: 16 x 4096 x 16384 points, a column
// launch 13 -> 10 us and a row launch 20 -> 12 us); each lane issues the loads
// of kSB of its pairs together before using them (kSBRev in the reverse row
// launches, whose pairs carry more registers: eight waves per SIMD). Sums are per
// lane in pair order, then a butterfly over the group, so results do not
// depend on scheduling.
constexpr int kSG = 4;
constexpr int kSB = 8;
constexpr int kSBRev = 4;

// Both sides' first scalings.
__global__ __launch_bounds__(kBlock) void k_fill_ones(DevPlan d)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int BN = d.B * d.N, BM = d.B * d.M;
    if (k < BN)
        d.alpha[k] = 1.0;
    if (k < BM)
        d.beta[k] = 1.0;
}

// Sum over an owner's pairs k = lg, lg + G, ... of f(k, position) with the
// loads of SB pairs in flight at once, added up over its G lanes.
template <int SB = kSB, class Load, class Use>
__device__ __forceinline__ double owner_sum(int n, int G, int lg, Load load, Use use)
{
    double acc = 0.0;
    for (int k0 = lg; k0 < n; k0 += G * SB) {
        decltype(load(0)) v[SB];
#pragma unroll
        for (int u = 0; u < SB; ++u)
            v[u] = load(k0 + G * u < n ? k0 + G * u : -1);
#pragma unroll
        for (int u = 0; u < SB; ++u)
            if (k0 + G * u < n)
                acc += use(v[u]);
    }
    return group_sum(acc, G);
}

// Column step (Eq. 3, COL) or row step (Eq. 4) of iteration l for all owners.
template <bool COL>
__device__ __forceinline__ void sink_owner(const DevPlan &d, int l, double eps, int o, int G, int lg)
{
    const int n_own = COL ? d.M : d.N, n_oth = COL ? d.N : d.M;
    const int b = o / n_own;
    const size_t BN = (size_t)d.B * d.N, BM = (size_t)d.B * d.M;
    const int32_t *ptr = COL ? d.col_ptr : d.row_ptr;
    const int32_t *idx = COL ? d.csc_row : d.csr_col;
    const float *p0 = COL ? d.p0c : d.p0r;
    // the other side's scalings: alpha^(l-1) for columns, beta^l for rows
    const double *oth = (COL ? d.alpha + (size_t)(l - 1) * BN : d.beta + (size_t)l * BM) + (size_t)b * n_oth;
    double *cur = COL ? d.beta : d.alpha;
    const size_t BO = COL ? BM : BN;
    const double prev = cur[(size_t)(l - 1) * BO + o]; // loaded with the segment bounds
    const int s0 = ptr[o], n = ptr[o + 1] - s0;
    struct V {
        float p;
        double x;
    };
    const double acc = owner_sum(n, G, lg,
                                 [&](int k) {
                                     V v{0.0f, 0.0};
                                     if (k >= 0) {
                                         v.p = p0[s0 + k];
                                         v.x = oth[idx[s0 + k]];
                                     }
                                     return v;
                                 },
                                 [&](const V &v) { return (double)v.p * v.x; });
    if (lg == 0) {
        const double den = prev * acc + eps;
        cur[(size_t)l * BO + o] = prev / den;
    }
}

template <bool COL, int G> __global__ __launch_bounds__(kBlock) void k_sink_step(DevPlan d, int l, double eps)
{
    // each XCD takes a contiguous range of owners: its L2 holds only the
    // other side's scalings of those owners' samples
    const int gid = xcd_contiguous(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    each_owner<kSB>(G, gid / G, d.B * (COL ? d.M : d.N), COL ? d.col_ptr : d.row_ptr,
                       [&](int lanes, int o, int lg) { sink_owner<COL>(d, l, eps, o, lanes, lg); });
}

__device__ __forceinline__ void loss_row(const DevPlan &d, double *loss_rows, int r, int G, int lg)
{
    const int b = r / d.N;
    const size_t BN = (size_t)d.B * d.N, BM = (size_t)d.B * d.M;
    const double *beta = d.beta + (size_t)d.L * BM + (size_t)b * d.M;
    const int t0 = d.row_ptr[r], n = d.row_ptr[r + 1] - t0;
    struct V {
        float p;
        double bc;
    };
    const double acc = owner_sum(n, G, lg,
                                 [&](int k) {
                                     V v{0.0f, 0.0};
                                     if (k >= 0) {
                                         v.p = d.p0r[t0 + k];
                                         v.bc = beta[d.csr_col[t0 + k]] * d.cost[t0 + k];
                                     }
                                     return v;
                                 },
                                 [&](const V &v) { return (double)v.p * v.bc; });
    if (lg == 0)
        loss_rows[r] = d.alpha[(size_t)d.L * BN + r] * acc;
}

template <int G> __global__ __launch_bounds__(kBlock) void k_loss_rows(DevPlan d, double *loss_rows)
{
    const int gid = xcd_contiguous(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; // as in k_sink_step
    each_owner<kSB>(G, gid / G, d.B * d.N, d.row_ptr,
                       [&](int lanes, int r, int lg) { loss_row(d, loss_rows, r, lanes, lg); });
}

// Per sample: the sum of its row losses. 1024 threads, four partial sums per
// thread so that four loads are in flight; fixed association.
constexpr int kLossT = 1024;

__global__ __launch_bounds__(kLossT) void k_loss_reduce(DevPlan d, const double *loss_rows)
{
    __shared__ double part[kLossT / 64];
    const int b = blockIdx.x;
    const double *lr = loss_rows + (size_t)b * d.N;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i0 = threadIdx.x; i0 < d.N; i0 += 4 * kLossT)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u * kLossT < d.N)
                s[u] += lr[i0 + u * kLossT];
    double t = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
    if (lane_id() == 0)
        part[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0;
        for (int w = 0; w < kLossT / 64; ++w)
            a += part[w];
        d.loss[b] = (float)a;
    }
}

// Reverse sweeps, one launch per half-step, on the owners' scalings alone.
// With f(c, s) = c / (c s + eps), df/dc = eps (f / c)^2 and df/ds = -f^2, so
// the adjoints of the row and column sums of P0 against the other side's
// scalings,
//   Rbar^l_i = -(alpha^l_i)^2 alphabar^l_i   (of sum_j P0_ij beta^l_j),
//   Sbar^l_j = -(beta^l_j)^2 betabar^l_j     (of sum_i alpha^(l-1)_i P0_ij),
// follow one another without any per-pair state:
//   Sbar^l_j     = eps Sbar^(l+1)_j - (beta^l_j)^2 sum_i P0_ij Rbar^l_i
//   Rbar^(l-1)_i = eps Rbar^l_i - (alpha^(l-1)_i)^2 sum_j P0_ij Sbar^l_j
// (a factor of a square at a time: with N != M alpha and beta drift by N / M an
// iteration, and where they pass 1e154 the square itself leaves the range of a
// double while the terms stay near the other side's scale)
// from the direct terms of the loss (sum alpha^L P0 beta^L C; k_bwd_direct), and
//   dLoss/dP0_ij = g alpha^L_i beta^L_j C_ij
//                  + sum_l (Rbar^l_i beta^l_j + alpha^(l-1)_i Sbar^l_j),
// whose sum the row launches form in row order, in double precision (adj; the
// softmax adjoints add the direct term). A column
// launch reads 16 bytes a pair (P0, index, Rbar), a row launch 40 (P0, index,
// the pair's sum, and beta, Sbar in one gather). With the adjoint itself kept
// per pair, once in each order, both launches moved 56: per launch 23 -> 11 us
// (columns) and 33 -> 19 us (rows) at 16 x 4096 x 16384 points, 21 -> 12 and
// 23 -> 14 us at 4 x 65536.
//
// The first adjoints of the reverse sweeps, all owners in one launch (rows
// first): Rbar^L_i = -(alpha^L_i)^2 g sum_j P0_ij beta^L_j C_ij into rbar and the
// same of the columns, the direct term of Sbar^L_j, into cs.
template <bool COL> __device__ __forceinline__ void direct_owner(const DevPlan &d, int o, int G, int lg)
{
    const int n_own = COL ? d.M : d.N, n_oth = COL ? d.N : d.M;
    const int b = o / n_own;
    const size_t BN = (size_t)d.B * d.N, BM = (size_t)d.B * d.M;
    const double *oth = (COL ? d.alpha + (size_t)d.L * BN : d.beta + (size_t)d.L * BM) + (size_t)b * n_oth;
    const double own = COL ? d.beta[(size_t)d.L * BM + o] : d.alpha[(size_t)d.L * BN + o], gl = d.grad_loss[b];
    const int32_t *ptr = COL ? d.col_ptr : d.row_ptr, *idx = COL ? d.csc_row : d.csr_col;
    const float *p0 = COL ? d.p0c : d.p0r;
    const int s0 = ptr[o], n = ptr[o + 1] - s0;
    struct V {
        double x, c;
        float p;
    };
    const double acc = owner_sum(n, G, lg,
                                 [&](int k) {
                                     V v{0.0, 0.0, 0.0f};
                                     if (k >= 0) {
                                         v.x = oth[idx[s0 + k]];
                                         v.c = d.cost[COL ? d.csc_perm[s0 + k] : s0 + k];
                                         v.p = p0[s0 + k];
                                     }
                                     return v;
                                 },
                                 [&](const V &v) { return (double)v.p * (v.x * v.c); });
    if (lg == 0) {
        const double first = -own * (own * (gl * acc));
        if (COL)
            d.cs[o] = make_double2(own, first);
        else
            d.rbar[o] = first;
    }
}

// Groups of GR lanes per row in the first row_blocks workgroups, of GC per column in the others.
__global__ __launch_bounds__(kBlock) void k_bwd_direct(DevPlan d, int row_blocks, int lr, int lc)
{
    const int bid = blockIdx.x;
    if (bid < row_blocks) {
        const int gid = xcd_contiguous(bid, row_blocks) * kBlock + threadIdx.x;
        each_owner<kSB>(1 << lr, gid >> lr, d.B * d.N, d.row_ptr,
                        [&](int lanes, int o, int lg) { direct_owner<false>(d, o, lanes, lg); });
    } else {
        const int gid = xcd_contiguous(bid - row_blocks, gridDim.x - row_blocks) * kBlock + threadIdx.x;
        each_owner<kSB>(1 << lc, gid >> lc, d.B * d.M, d.col_ptr,
                        [&](int lanes, int o, int lg) { direct_owner<true>(d, o, lanes, lg); });
    }
}

// Column launch l: Sbar^l. keep: the factor of the value in cs, 1 for the
// direct term (l = L), then eps.
__device__ __forceinline__ void bwd_col(const DevPlan &d, int l, double keep, int gc, int G, int lg)
{
    const int b = gc / d.M;
    const double *rbar = d.rbar + (size_t)b * d.N;
    const double bl = d.beta[(size_t)l * d.B * d.M + gc], old = keep * d.cs[gc].y;
    const int s0 = d.col_ptr[gc], n = d.col_ptr[gc + 1] - s0;
    struct V {
        float p;
        double x;
    };
    const double acc = owner_sum(n, G, lg,
                                 [&](int k) {
                                     V v{0.0f, 0.0};
                                     if (k >= 0) {
                                         v.p = d.p0c[s0 + k];
                                         v.x = rbar[d.csc_row[s0 + k]];
                                     }
                                     return v;
                                 },
                                 [&](const V &v) { return (double)v.p * v.x; });
    if (lg == 0)
        d.cs[gc] = make_double2(bl, old - bl * (bl * acc));
}

template <int G> __global__ __launch_bounds__(kBlock) void k_bwd_cols(DevPlan d, int l, double keep)
{
    const int gid = xcd_contiguous(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; // as in k_sink_step
    each_owner<kSB>(G, gid / G, d.B * d.M, d.col_ptr,
                    [&](int lanes, int gc, int lg) { bwd_col(d, l, keep, gc, lanes, lg); });
}

// Row launch after column launch l: the pairs' terms of iteration l, Rbar^(l-1).
// FIRST (l = L): the first terms.
template <bool FIRST>
__device__ __forceinline__ void bwd_row(const DevPlan &d, int l, double eps, int r, int G, int lg)
{
    const int b = r / d.N;
    const double2 *cs = d.cs + (size_t)b * d.M;
    const double rb = d.rbar[r], al = d.alpha[(size_t)(l - 1) * d.B * d.N + r];
    const int t0 = d.row_ptr[r], n = d.row_ptr[r + 1] - t0;
    struct V {
        double2 c;
        double z;
        float p;
        int k;
    };
    const double acc = owner_sum<kSBRev>(n, G, lg,
                                         [&](int k) {
                                             V v{make_double2(0.0, 0.0), 0.0, 0.0f, k};
                                             if (k >= 0) {
                                                 v.c = cs[d.csr_col[t0 + k]];
                                                 v.z = FIRST ? 0.0 : d.adj[t0 + k];
                                                 v.p = d.p0r[t0 + k];
                                             }
                                             return v;
                                         },
                                         [&](const V &v) {
                                             d.adj[t0 + v.k] =
                                                 __builtin_fma(rb, v.c.x, __builtin_fma(al, v.c.y, v.z));
                                             return v.c.y * (double)v.p;
                                         });
    if (lg == 0)
        d.rbar[r] = eps * rb - al * (al * acc);
}

template <bool FIRST, int G> __global__ __launch_bounds__(kBlock) void k_bwd_rows(DevPlan d, int l, double eps)
{
    const int gid = xcd_contiguous(blockIdx.x, gridDim.x) * kBlock + threadIdx.x; // as in k_sink_step
    each_owner<kSB>(G, gid / G, d.B * d.N, d.row_ptr,
                       [&](int lanes, int r, int lg) { bwd_row<FIRST>(d, l, eps, r, lanes, lg); });
}

} // namespace

int sinkhorn_slots(int N, int M, const int32_t *counts, int B)
{
    if (N > kSinkOwners || M > kSinkOwners)
        return 0;
    int most = 1;
    for (int b = 0; b < B; ++b) {
        if (counts[4 * b + 2] > kSinkMaxGroup || counts[4 * b + 3] > kSinkMaxGroup)
            return 0;
        most = std::max({most, counts[4 * b], counts[4 * b + 1]});
    }
    const int slots = (most + kT - 1) / kT;
    return slots <= kSinkMaxSlots ? slots : 0;
}

int sinkhorn_slots_wide(int N, int M, const int32_t *counts, int B)
{
    if (N > kSinkOwnersW || M > kSinkOwnersW)
        return 0;
    int most = 1;
    for (int b = 0; b < B; ++b) {
        if (counts[4 * b + 2] > kSinkMaxGroup || counts[4 * b + 3] > kSinkMaxGroup)
            return 0;
        most = std::max({most, counts[4 * b], counts[4 * b + 1]});
    }
    const int slots = (most + kT - 1) / kT;
    return slots <= kSinkMaxSlotsW ? slots : 0;
}

void launch_wide_pack(const DevPlan &d, int32_t *place, hipStream_t s)
{
    hipLaunchKernelGGL(k_place_w, dim3(d.B, 2), dim3(kT), 0, s, d, place);
    hipLaunchKernelGGL(k_pack_w, dim3(blocks_for(2 * d.nnz, kBlock)), dim3(kBlock), 0, s, d, (const int32_t *)place);
}

int sinkhorn_split_factor(int B)
{
    const char *env = std::getenv("APML_SINKHORN_SPLIT");
    if (env && env[0] == '0')
        return 1;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64 || B < 1)
        return 1;
    // workgroups of the split kernels resident at once on each device, plus 1
    // (0: not yet queried)
    static std::atomic<int> resident[64];
    int c = resident[dev].load(std::memory_order_relaxed);
    if (c == 0) {
        int cus = 0, coop = 0, f = 0, r = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&f, reinterpret_cast<const void *>(k_sinkhorn_fwd_ws), kT, 0) !=
                hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, reinterpret_cast<const void *>(k_sinkhorn_bwd_ws), kT, 0) !=
                hipSuccess) {
            (void)hipGetLastError();
            cus = coop = 0;
        }
        c = (coop ? cus * std::min(f, r) : 0) + 1;
        resident[dev].store(c, std::memory_order_relaxed);
    }
    // the grid rounds B up to whole rounds of the eight XCDs
    const int K = std::min(kSplitMax, (c - 1) / split_grid(B, 1));
    return K >= 2 ? K : 1;
}

namespace {

// Clears the sample's meeting counters, then launches the split kernel over
// B K workgroups, all resident at once; false when the cooperative launch
// is refused (the caller then takes the one-workgroup kernel).
bool launch_split(const void *kernel, void **args, const DevPlan &d, int K, size_t lds, hipStream_t s)
{
    const int n = d.B * 2 * kSplitSyncStride;
    hipLaunchKernelGGL(k_zero_u32, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, d.split_sync, n);
    if (hipGetLastError() != hipSuccess)
        return false;
    if (hipLaunchCooperativeKernel(kernel, dim3(split_grid(d.B, K)), dim3(kT), args, lds, s) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return true;
}

// APML_SINKHORN_SPLIT=streamed keeps the split kernels but takes their
// streamed variants at any share (the variants give the same bits; this
// lets them be compared).
bool split_streamed_only()
{
    const char *env = std::getenv("APML_SINKHORN_SPLIT");
    return env && env[0] == 's';
}

// The split kernel for a workgroup share of sw slots per lane and order:
// registers up to the limit, else streamed.
const void *split_fwd_kernel(int sw)
{
    if (split_streamed_only())
        return reinterpret_cast<const void *>(k_sinkhorn_fwd_ws);
    switch (sw) {
    case 1: return reinterpret_cast<const void *>(k_sinkhorn_fwd_wr<1>);
    case 2: return reinterpret_cast<const void *>(k_sinkhorn_fwd_wr<2>);
    case 3: return reinterpret_cast<const void *>(k_sinkhorn_fwd_wr<3>);
    default: return reinterpret_cast<const void *>(k_sinkhorn_fwd_ws);
    }
}

const void *split_bwd_kernel(int sw)
{
    if (split_streamed_only())
        return reinterpret_cast<const void *>(k_sinkhorn_bwd_ws);
    switch (sw) {
    case 1: return reinterpret_cast<const void *>(k_sinkhorn_bwd_wr<1>);
    case 2: return reinterpret_cast<const void *>(k_sinkhorn_bwd_wr<2>);
    case 3: return reinterpret_cast<const void *>(k_sinkhorn_bwd_wr<3>);
    case 4: return reinterpret_cast<const void *>(k_sinkhorn_bwd_wr<4>);
    default: return reinterpret_cast<const void *>(k_sinkhorn_bwd_ws);
    }
}

static_assert(kSplitRegFwd == 3 && kSplitRegBwd == 4, "instances above");

} // namespace

hipError_t launch_sinkhorn_fwd_wide(const DevPlan &d, double eps, hipStream_t s)
{
    // a forward half-sweep over fewer slots is shorter than the meeting that
    // splitting it needs (measured: 3000 to 4096 points per cloud, 4 to 6
    // slots, 0.09 -> 0.13 ms; 10 to 12 slots: 37 x 7000 points 0.185 -> 0.135 ms,
    // 72 x 8000 0.257 -> 0.236)
    constexpr int kSplitFwdMinSlots = 8;
    int K = d.wk_row.slots >= kSplitFwdMinSlots ? sinkhorn_split_factor(d.B) : 1;
    if (K > 1 && d.split_sync) {
        DevPlan dc = d;
        double e = eps;
        void *args[] = {&dc, &e, &K};
        if (launch_split(split_fwd_kernel((d.wk_row.slots + K - 1) / K), args, d, K, 0, s))
            return hipSuccess;
    }
    hipLaunchKernelGGL(k_sinkhorn_fwd_w, dim3(d.B), dim3(kT), 0, s, d, eps);
    return hipGetLastError();
}

bool sinkhorn_bwd_streams(int slots, int B)
{
    const int K = sinkhorn_split_factor(B);
    return split_bwd_kernel((slots + K - 1) / K) == reinterpret_cast<const void *>(k_sinkhorn_bwd_ws);
}

size_t sinkhorn_exchange_words(int L, size_t owners) { return (size_t)L * phase_region(owners) + kSinkOwnersW; }

hipError_t launch_sinkhorn_bwd_wide(const DevPlan &d, double eps, hipStream_t s)
{
    int K = sinkhorn_split_factor(d.B);
    const int sw = (d.wk_row.slots + K - 1) / K;
    const void *kernel = split_bwd_kernel(sw);
    const bool streamed = kernel == reinterpret_cast<const void *>(k_sinkhorn_bwd_ws);
    const size_t lds = streamed ? 0 : 4 * (size_t)bwd_wide_lds_slots(sw) * kColSlotWords * kT;
    hipError_t err = set_dynamic_lds(kernel, lds);
    if (err != hipSuccess)
        return err;
    DevPlan dc = d;
    double e = eps;
    void *args[] = {&dc, &e, &K};
    if (K == 1) { // nothing to meet with (register kernels: 136 x 2100 points 233 us streamed, 157)
        err = hipLaunchKernel(kernel, dim3(split_grid(d.B, 1)), dim3(kT), args, lds, s);
        return err != hipSuccess ? err : hipGetLastError();
    }
    if (!launch_split(kernel, args, d, K, lds, s)) // the cooperative launch was refused
        launch_sinkhorn_bwd_steps(d, eps, s);
    return hipGetLastError();
}

size_t packed_order_words(int B, int slots) { return (size_t)B * slots * kP * kT; }

void launch_place(const DevPlan &d, int32_t *place, hipStream_t s)
{
    hipLaunchKernelGGL(k_place, dim3(d.B, 2), dim3(kT), 0, s, d, place);
}

// The kernel instance for the plan's slot count.
template <template <int> class K> static auto for_slots(int slots) -> decltype(K<1>::fn)
{
    switch (slots) {
    case 1: return K<1>::fn;
    case 2: return K<2>::fn;
    case 3: return K<3>::fn;
    case 4: return K<4>::fn;
    case 5: return K<5>::fn;
    default: return K<6>::fn;
    }
}
template <int S> struct FwdK { static constexpr auto fn = k_sinkhorn_fwd<S>; };
template <int S> struct BwdK { static constexpr auto fn = k_sinkhorn_bwd<S>; };

hipError_t launch_sinkhorn_fwd(const DevPlan &d, double eps, hipStream_t s)
{
    const auto k = for_slots<FwdK>(d.pk_row.slots);
    hipLaunchKernelGGL(k, dim3(d.B), dim3(kT), 0, s, d, eps);
    return hipGetLastError();
}

hipError_t launch_sinkhorn_bwd(const DevPlan &d, double eps, hipStream_t s)
{
    const size_t bytes = 4 * (size_t)bwd_lds_slots(d.pk_row.slots) * kColSlotWords * kT; // beyond the static arrays
    const auto k = for_slots<BwdK>(d.pk_row.slots);
    hipError_t e = set_dynamic_lds((const void *)k, bytes);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k, dim3(d.B), dim3(kT), bytes, s, d, eps);
    return hipGetLastError();
}

namespace {

// Lanes per owner of the per-iteration kernels: the largest power of two
// up to the owners' mean pair count, within 4..16 (rows of 18 pairs on
// average: 16 lanes took the sweeps of the unequal workload from 0.38 / 0.79
// ms to 0.29 / 0.61 ms; at 5 pairs, 4 lanes stay the fastest).
int steps_lanes(int64_t nnz, int64_t owners)
{
    int g = kSG;
    while (g < 16 && (int64_t)g * 2 * owners <= nnz)
        g *= 2;
    return g;
}

int log2_lanes(int g) { return g == 16 ? 4 : g == 8 ? 3 : 2; }

template <template <int> class K, class... A>
void launch_lanes(int g, int64_t owners, hipStream_t s, A... args)
{
    switch (g) {
    case 8: hipLaunchKernelGGL(K<8>::fn, dim3(blocks_for(owners * 8, kBlock)), dim3(kBlock), 0, s, args...); break;
    case 16: hipLaunchKernelGGL(K<16>::fn, dim3(blocks_for(owners * 16, kBlock)), dim3(kBlock), 0, s, args...); break;
    default: hipLaunchKernelGGL(K<4>::fn, dim3(blocks_for(owners * 4, kBlock)), dim3(kBlock), 0, s, args...); break;
    }
}
template <int G> struct ColStep { static constexpr auto fn = k_sink_step<true, G>; };
template <int G> struct RowStep { static constexpr auto fn = k_sink_step<false, G>; };
template <int G> struct BwdRowsFirst { static constexpr auto fn = k_bwd_rows<true, G>; };
template <int G> struct BwdRows { static constexpr auto fn = k_bwd_rows<false, G>; };
template <int G> struct BwdCols { static constexpr auto fn = k_bwd_cols<G>; };
template <int G> struct LossRows { static constexpr auto fn = k_loss_rows<G>; };

} // namespace

void launch_bwd_direct(const DevPlan &d, hipStream_t s)
{
    const int64_t BN = (int64_t)d.B * d.N, BM = (int64_t)d.B * d.M;
    const int gr = steps_lanes(d.nnz, BN), gc = steps_lanes(d.nnz, BM);
    const unsigned rows = blocks_for(BN * gr, kBlock), cols = blocks_for(BM * gc, kBlock);
    hipLaunchKernelGGL(k_bwd_direct, dim3(rows + cols), dim3(kBlock), 0, s, d, (int)rows, log2_lanes(gr), log2_lanes(gc));
}

void launch_sinkhorn_fwd_steps(const DevPlan &d, double eps, hipStream_t s)
{
    const int BN = d.B * d.N, BM = d.B * d.M;
    const int gr = steps_lanes(d.nnz, BN), gc = steps_lanes(d.nnz, BM);
    hipLaunchKernelGGL(k_fill_ones, dim3(blocks_for(std::max(BN, BM), kBlock)), dim3(kBlock), 0, s, d);
    for (int l = 1; l <= d.L; ++l) {
        launch_lanes<ColStep>(gc, BM, s, d, l, eps);
        launch_lanes<RowStep>(gr, BN, s, d, l, eps);
    }
    // the backward scratch is free during the forward pass: use it for the row losses
    launch_lanes<LossRows>(gr, BN, s, d, d.dvec);
    hipLaunchKernelGGL(k_loss_reduce, dim3(d.B), dim3(kLossT), 0, s, d, (const double *)d.dvec);
}

void launch_sinkhorn_bwd_steps(const DevPlan &d, double eps, hipStream_t s)
{
    const int BN = d.B * d.N, BM = d.B * d.M;
    const int gr = steps_lanes(d.nnz, BN), gc = steps_lanes(d.nnz, BM);
    for (int l = d.L; l >= 1; --l) {
        launch_lanes<BwdCols>(gc, BM, s, d, l, l == d.L ? 1.0 : eps);
        if (l == d.L)
            launch_lanes<BwdRowsFirst>(gr, BN, s, d, l, eps);
        else
            launch_lanes<BwdRows>(gr, BN, s, d, l, eps);
    }
}

} // namespace apml
