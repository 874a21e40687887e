// Device helpers shared by the libapml kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>

namespace apml {

constexpr float kInf = __builtin_huge_valf();

// Squared distance in single precision, as d = a - b per coordinate, then
// dx*dx, fma(dy,dy,.), fma(dz,dz,.). The dense scans and the sparse passes
// evaluate exactly this sequence (the library is built without floating-point
// contraction), so their values agree bit for bit; the argmin decisions rest
// on it.
__device__ __forceinline__ float sqdist_f32(float ax, float ay, float az, float bx, float by,
                                            float bz)
{
    const float dx = ax - bx, dy = ay - by, dz = az - bz;
    float s = dx * dx;
    s = __builtin_fmaf(dy, dy, s);
    s = __builtin_fmaf(dz, dz, s);
    return s;
}

// Cost C = ||a - b||_2 (Sec. III-A) in double precision from float coordinates.
__device__ __forceinline__ double dist_f64(const float *a, const float *b)
{
    const double dx = (double)a[0] - (double)b[0];
    const double dy = (double)a[1] - (double)b[1];
    const double dz = (double)a[2] - (double)b[2];
    return sqrt(dx * dx + dy * dy + dz * dz);
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// Number of entries of a[s0, s1) below key: sixteen loads in flight at a time,
// then four (a loop of one load per step waits out every load in turn).
__device__ __forceinline__ int count_below(const int32_t *a, int s0, int s1, int key)
{
    int n = 0, q = s0;
    for (; q + 16 <= s1; q += 16) {
        int v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            v[u] = a[q + u];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            n += v[u] < key;
    }
    for (; q + 4 <= s1; q += 4) {
        const int v0 = a[q], v1 = a[q + 1], v2 = a[q + 2], v3 = a[q + 3];
        n += (v0 < key) + (v1 < key) + (v2 < key) + (v3 < key);
    }
    for (; q < s1; ++q)
        n += a[q] < key;
    return n;
}

// Read-only data seen through the constant address space: wave-uniform loads
// from it become scalar loads even in kernels that also store to memory.
template <typename T> using const_ptr = const __attribute__((address_space(4))) T *;
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename T> __device__ __forceinline__ const_ptr<T> as_const(const T *p)
{
    return (const_ptr<T>)p;
}

// Reductions over aligned groups of G lanes (G divides 64). Butterfly order:
// every lane of a group ends with the same, order-independent bits.
template <int G> __device__ __forceinline__ double group_sum(double v)
{
#pragma unroll
    for (int o = 1; o < G; o <<= 1)
        v += __shfl_xor(v, o);
    return v;
}

// v from the partner lane of butterfly step K. Steps 0 and 1 pair lane i with
// i ^ 1 and i ^ 2 (quad_perm); from step 2 on, all lanes of an aligned block
// of 2^K lanes already hold the same value, so any lane of the neighbouring
// block will do: step 2 uses row_half_mirror (i -> 7 - i within 8), step 3
// row_mirror (i -> 15 - i within 16), both DPP moves; steps 4 and 5 use lane
// permutes across rows.
template <int K> __device__ __forceinline__ int partner(int v)
{
    if constexpr (K == 0)
        return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true); // quad_perm [1,0,3,2]
    else if constexpr (K == 1)
        return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true); // quad_perm [2,3,0,1]
    else if constexpr (K == 2)
        return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true); // row_half_mirror
    else if constexpr (K == 3)
        return __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true); // row_mirror
    else
        return __shfl_xor(v, 1 << K);
}
template <int K> __device__ __forceinline__ double partner(double v)
{
    int2 w = __builtin_bit_cast(int2, v);
    w.x = partner<K>(w.x);
    w.y = partner<K>(w.y);
    return __builtin_bit_cast(double, w);
}

// Reductions over aligned groups of G lanes, G a wave-uniform run-time power
// of two from 4 to 64.
__device__ __forceinline__ double group_sum(double v, int G)
{
    v += partner<0>(v);
    v += partner<1>(v);
    if (G > 4)
        v += partner<2>(v);
    if (G > 8)
        v += partner<3>(v);
    if (G > 16)
        v += partner<4>(v);
    if (G > 32)
        v += partner<5>(v);
    return v;
}

__device__ __forceinline__ int group_min(int v, int G)
{
    v = min(v, partner<0>(v));
    v = min(v, partner<1>(v));
    if (G > 4)
        v = min(v, partner<2>(v));
    if (G > 8)
        v = min(v, partner<3>(v));
    if (G > 16)
        v = min(v, partner<4>(v));
    if (G > 32)
        v = min(v, partner<5>(v));
    return v;
}

__device__ __forceinline__ double wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o);
    return v;
}

// Workgroup barrier that orders LDS accesses only: global stores issued
// before it may still be in flight (use __syncthreads when other threads of
// the workgroup read them back).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Barrier for a workgroup that shares data through LDS (LDS_ONLY) or also
// through global memory.
template <bool LDS_ONLY> __device__ __forceinline__ void wg_barrier()
{
    if (LDS_ONLY)
        lds_barrier();
    else
        __syncthreads();
}

// Calls f(lanes, owner, lane of the group) for the owner of each group of G
// lanes (a power of two from 4 to 64), then, for the owners whose segment exceeds
// CAP pairs a lane (what a lane loads at once), with the whole wave, one such
// owner after another.
// A group strides through a long segment with two dependent loads a step
// while the other groups of its wave wait: one point far from the rest keeps
// hundreds of candidates (its gap sets its radius), and its row alone took
// most of a launch. The lane count is a run-time value so that both uses
// share one copy of f: for short f (the sweeps); split_owners keeps two.
template <int CAP, class F> __device__ __forceinline__ void each_owner(int G, int o, int n_own, const int32_t *ptr, F f)
{
    const int n = o < n_own ? ptr[o + 1] - ptr[o] : 0;
    const bool spread = n > G * CAP;
    uint64_t left = __ballot(spread && (threadIdx.x & (G - 1)) == 0);
    bool mine = o < n_own && !spread;
    int lanes = G, lane = (int)(threadIdx.x & (G - 1)), owner = o;
    for (;;) {
        asm volatile("" : "+s"(lanes)); // one copy of f: the first pass is not peeled off
        if (mine)
            f(lanes, owner, lane);
        if (left == 0)
            break;
        owner = __builtin_amdgcn_readlane(o, __builtin_ctzll(left));
        left &= left - 1;
        lanes = 64;
        lane = lane_id();
        mine = true;
    }
}

// use(load(k), k) for k = k0, k0 + step, ... below n, SB loads in flight at a
// time (load must not depend on what use writes).
template <int SB, class Load, class Use>
__device__ __forceinline__ void strided(int k0, int n, int step, Load load, Use use)
{
    for (int k = k0; k < n; k += step * SB) {
        decltype(load(0)) v[SB];
#pragma unroll
        for (int u = 0; u < SB; ++u)
            v[u] = load(min(k + u * step, n - 1));
#pragma unroll
        for (int u = 0; u < SB; ++u)
            if (k + u * step < n)
                use(v[u], k + u * step);
    }
}

// Finds, among the pairs of one segment, the first position whose
// single-precision squared distance equals m1 and the first other position
// whose distance equals m2 (the second order statistic): the minimum and the
// second minimum with ties to the smaller index.
struct Argmins {
    int f1 = INT_MAX, g1 = INT_MAX, g2 = INT_MAX;
    __device__ void see(int t, float s, float2 m)
    {
        if (s == m.x && f1 == INT_MAX)
            f1 = t;
        if (s == m.y) {
            if (g1 == INT_MAX)
                g1 = t;
            else if (g2 == INT_MAX)
                g2 = t;
        }
    }
    __device__ void resolve(int *q1, int *q2, int G) const
    {
        *q1 = group_min(f1, G);
        *q2 = group_min(g1 != *q1 ? g1 : g2, G);
    }
};

// Workgroups are dealt to the 8 XCDs round robin (workgroup i to XCD i % 8),
// and each XCD has its own L2. This maps the hardware index to a logical one
// under which every XCD receives one contiguous range of the grid, so that
// workgroups sharing data (one sample) share an L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_contiguous(int bid, int grid)
{
    const int q = grid / kXcds, r = grid % kXcds, x = bid % kXcds;
    return x * q + min(x, r) + bid / kXcds;
}

// The owners of a launch in two kinds of workgroups of T threads. The first
// long_blocks take the owners of more than CAP pairs a lane of G, a wave each:
// wave w of W looks at owners w, w + W, ..., so that long ones that stand
// together (points repeated at a cloud's end) go to different waves. The others
// call shorter(owner, lane of the group) for the rest, in groups of G lanes. As
// two kinds the short owners' code keeps its compile-time lane count and carries
// none of the loops of the long ones'.
template <int G, int CAP, int T, class Short, class Long>
__device__ __forceinline__ void split_owners(int block, int blocks, int long_blocks, int n_own, const int32_t *ptr,
                                             Short shorter, Long longer)
{
    if (block < long_blocks) {
        const int waves = long_blocks * (T / 64), w = block * (T / 64) + ((int)threadIdx.x >> 6), lane = lane_id();
        for (int base = w; base < n_own; base += 64 * waves) {
            const int o = min(base + lane * waves, n_own); // owners stay below 2^29, waves below 2^12
            uint64_t left = __ballot(o < n_own && ptr[o + 1] - ptr[o] > G * CAP);
            for (; left; left &= left - 1)
                longer(base + __builtin_ctzll(left) * waves, lane);
        }
        return;
    }
    const int gid = xcd_contiguous(block - long_blocks, blocks - long_blocks) * T + (int)threadIdx.x;
    const int o = gid / G; // a sample's owners share an L2
    if (o < n_own && ptr[o + 1] - ptr[o] <= G * CAP)
        shorter(o, gid % G);
}

inline unsigned blocks_for(int64_t n, int per_block) { return (unsigned)((n + per_block - 1) / per_block); }

} // namespace apml
