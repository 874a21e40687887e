// Spatial order of the two clouds for the dense scans.
//
// Every pair whose distance can matter to a row or a column lies within a
// small radius (the kept ball of Sec. III-B, Eq. 1, or the second minimum of
// Sec. III-A). With each cloud sorted along a Hilbert curve, a run of 32
// consecutive points occupies a small box, and the dense scans skip every
// run whose box is provably beyond that radius from the box of their rows
// (dense.hip). The order only decides which work is skipped: results do not
// depend on it.
//
//   k_sort_frame    partial bounding cubes of both clouds of a sample.
//   k_spatial_sort  one workgroup per (sample, cloud, chunk of 2048 points).
//                   The bounding cube is quantized to 10 bits per axis; the
//                   upper 20 bits of the 30-bit Hilbert keys are sorted by a
//                   least-significant-digit radix sort (two 10-bit digits,
//                   stable: ranks within a wave from ballots, across waves
//                   from per-wave digit counts in LDS).
//   k_sort_merge    up to 16 sorted runs merged at once, one level per launch:
//                   each element's place is its own index plus its rank in
//                   every other run.
//   k_sort_gather   the sorted points as (x, y, z, original index), the
//                   bounding box of every run of 32 and of every batch of 64
//                   runs.
#include <algorithm>

#include "apml_internal.h"
#include "device_common.h"

namespace apml {
namespace {

constexpr int kSortT = 1024;
constexpr int kSortWaves = kSortT / 64;
constexpr int kDigitBits = 10;
constexpr int kBins = 1 << kDigitBits; // == kSortT: one bin per thread in the scans
constexpr int kPasses = 3;
constexpr int kFirstPass = 1; // the lowest digit is not sorted (see k_spatial_sort)
constexpr int kSuper = 2; // keys per thread, in registers
// Points sorted by one workgroup; a cloud is sorted in chunks of this many
// points in parallel, and the chunks are then merged. A workgroup's tiles of
// 1024 keys follow each other through four barriers each, so few points per
// workgroup and more of them: 20000 + 20000 points 16.5 us, in chunks of 8192
// 51 us.
constexpr int kSortChunk = kSuper * kSortT;
// Chunks merged at once: every element of a merge finds its place in the
// other chunks by binary searches that don't depend on each other, so one
// level of many chunks costs little more than one of two.
constexpr int kMergeWays = 16;
static_assert(kBins == kSortT, "one bin per thread");
static_assert(kSortChunk == 64 * kRun, "a workgroup's points are one batch of runs");

// Spreads the low 10 bits of v to every third bit (bit k goes to bit 3k).
__device__ __forceinline__ uint32_t spread3(uint32_t v)
{
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Position along the Hilbert curve of the cell (x, y, z), 10 bits per axis,
// by Skilling's transposition ("Programming the Hilbert curve", 2004): the
// axes are turned into the transposed Hilbert index, whose bits interleaved
// give the 30-bit key. Consecutive keys are adjacent cells, so a run of
// consecutive points stays compact (a Morton order jumps across the space).
__device__ __forceinline__ uint32_t hilbert_key(uint32_t x, uint32_t y, uint32_t z)
{
    uint32_t X[3] = {x, y, z};
#pragma unroll
    for (uint32_t Q = 1u << 9; Q > 1; Q >>= 1) {
        const uint32_t P = Q - 1;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (X[i] & Q) {
                X[0] ^= P; // invert the low bits of the first axis
            } else {       // exchange the low bits of the first axis and axis i
                const uint32_t t = (X[0] ^ X[i]) & P;
                X[0] ^= t;
                X[i] ^= t;
            }
        }
    }
    X[1] ^= X[0]; // Gray encode
    X[2] ^= X[1];
    uint32_t t = 0;
#pragma unroll
    for (uint32_t Q = 1u << 9; Q > 1; Q >>= 1)
        if (X[2] & Q)
            t ^= Q - 1;
    X[0] ^= t;
    X[1] ^= t;
    X[2] ^= t;
    return spread3(X[2]) | spread3(X[1]) << 1 | spread3(X[0]) << 2;
}

__device__ __forceinline__ uint32_t quantize(float v, float lo, float scale)
{
    const float t = (v - lo) * scale;
    return (uint32_t)fminf(fmaxf(t, 0.0f), 1023.0f);
}

// LDS of k_spatial_sort (dynamic; about 156 KB).
struct SortLds {
    int whist[kSortWaves][kBins]; // digit counts of each wave in the current tile (zero outside a tile)
    int woff[kSortWaves][kBins];  // their exclusive prefix over the waves
    int base[kPasses - kFirstPass][kBins]; // next output position of every digit, per pass
    uint2 mid[kSortChunk];        // keys and values between the passes
    int wsum[kSortWaves];
};

__device__ __forceinline__ uint64_t lanes_below() { return (1ull << lane_id()) - 1ull; }

// One stable pass: put(position, key, value) of the n keys of the workgroup,
// key u * kSortT + tid of thread tid, in order of digit pass p.
template <class Put>
__device__ __forceinline__ void radix_pass(SortLds &s, int p, int n, const uint32_t (&key)[kSuper],
                                           const uint32_t (&val)[kSuper], Put put)
{
    const int tid = threadIdx.x, wave = tid >> 6;
    const int shift = p * kDigitBits;
    int *base = s.base[p - kFirstPass];
#pragma unroll
    for (int u = 0; u < kSuper; ++u) {
        const int k0 = u * kSortT;
        if (k0 >= n) // uniform over the workgroup
            break;
        const bool valid = k0 + tid < n;
        const uint32_t dg = (key[u] >> shift) & (kBins - 1);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int i = 0; i < kDigitBits; ++i) {
            const uint64_t bal = __ballot((dg >> i) & 1u);
            peers &= ((dg >> i) & 1u) ? bal : ~bal;
        }
        const uint64_t lower = peers & lanes_below();
        const int rank = __popcll(lower);
        const bool leader = valid && lower == 0;
        if (leader)
            s.whist[wave][dg] = __popcll(peers);
        lds_barrier();
        int run = 0;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            const int c = s.whist[w][tid];
            s.woff[w][tid] = run;
            run += c;
        }
        lds_barrier();
        const int pos = base[dg] + s.woff[wave][dg] + rank;
        if (valid && pos < n) // always below n: every pass sees the digits the histograms counted
            put(pos, key[u], val[u]);
        lds_barrier();
        base[tid] += run;
        if (leader) // this wave's next tile writes its counts after these clears (same wave, in order)
            s.whist[wave][dg] = 0;
    }
    lds_barrier();
}

// Component-wise union of the boxes of the W lanes around this one.
template <int W>
__device__ __forceinline__ void union_box(float lo[3], float hi[3])
{
#pragma unroll
    for (int o = 1; o < W; o <<= 1)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lo[c] = fminf(lo[c], __shfl_xor(lo[c], o));
            hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], o));
        }
}

// Bounding box of points [k0, k1) of sample b, numbered over X then Y, into
// f (min x, y, z, max x, y, z; every thread of the workgroup gets it). wf:
// LDS for the per-wave boxes. Ends with an LDS barrier.
__device__ void frame_of(const SpatialArgs &a, int b, int k0, int k1, float f[6], float (*wf)[6])
{
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const float *xs = a.x + (size_t)b * a.N * 3, *ys = a.y + (size_t)b * a.M * 3;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        f[c] = kInf;
        f[3 + c] = -kInf;
    }
    for (int k = k0 + tid; k < k1; k += kSortT) {
        const float *p = k < a.N ? xs + 3 * (size_t)k : ys + 3 * (size_t)(k - a.N);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            f[c] = fminf(f[c], p[c]);
            f[3 + c] = fmaxf(f[3 + c], p[c]);
        }
    }
    union_box<64>(f, f + 3);
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < 6; ++c)
            wf[wave][c] = f[c];
    lds_barrier();
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            f[c] = fminf(f[c], wf[w][c]);
            f[3 + c] = fmaxf(f[3 + c], wf[w][3 + c]);
        }
}

// The partial box of one slice of a sample (both clouds), combined by every
// chunk of the sample: workgroup (sample, slice).
__global__ __launch_bounds__(kSortT) void k_sort_frame(SpatialArgs a)
{
    __shared__ float wf[kSortWaves][6];
    const int b = blockIdx.x / a.frame_slices, q = blockIdx.x % a.frame_slices, n = a.N + a.M;
    const int per = (n + a.frame_slices - 1) / a.frame_slices;
    float f[6];
    frame_of(a, b, q * per, min(n, (q + 1) * per), f, wf);
    if (threadIdx.x < 6)
        a.frame_part[((size_t)b * a.frame_slices + q) * 6 + threadIdx.x] = f[threadIdx.x];
}

__global__ __launch_bounds__(kSortT) void k_spatial_sort(SpatialArgs a)
{
    extern __shared__ int4 lds_raw[];
    SortLds &s = *reinterpret_cast<SortLds *>(lds_raw);
    // workgroup: (sample, cloud, chunk of kSortChunk points)
    const int chunks = (max(a.N, a.M) + kSortChunk - 1) / kSortChunk;
    const int c = blockIdx.x % chunks, b = blockIdx.x / chunks / 2, cloud = blockIdx.x / chunks % 2;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    if (blockIdx.x == 0 && tid < 2 * kScanSlots) {
        (&a.ctr->scanned[0][0])[tid] = 0;
        if (tid == 0) {
            a.ctr->error = 0;
            a.ctr->overflow = 0;
        }
    }
    const int n_all = cloud ? a.M : a.N;
    const int c0 = c * kSortChunk;
    if (c0 >= n_all) // this cloud has fewer chunks (uniform over the workgroup)
        return;
    const int n = min(kSortChunk, n_all - c0);
    const float *pts = (cloud ? a.y : a.x) + ((size_t)b * n_all + c0) * 3;
    const size_t seg = (cloud ? (size_t)a.B * a.pad_x + (size_t)b * a.pad_y : (size_t)b * a.pad_x) + c0;

    // frame: bounding cube of both clouds of the sample
    float f[6];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        f[c] = kInf;
        f[3 + c] = -kInf;
    }
    for (int q = lane; q < a.frame_slices; q += 64) {
        const float *v = a.frame_part + ((size_t)b * a.frame_slices + q) * 6;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            f[c] = fminf(f[c], v[c]);
            f[3 + c] = fmaxf(f[3 + c], v[3 + c]);
        }
    }
    union_box<64>(f, f + 3);
    for (int i = tid; i < (kPasses - kFirstPass) * kBins; i += kSortT)
        (&s.base[0][0])[i] = 0;
    for (int i = tid; i < kSortWaves * kBins; i += kSortT)
        (&s.whist[0][0])[i] = 0;
    lds_barrier();
    const float ext = fmaxf(fmaxf(f[3] - f[0], f[4] - f[1]), f[5] - f[2]);
    const float scale = ext > 0.0f ? 1024.0f / ext : 0.0f;

    // keys and the digit histograms of the passes (independent of the order).
    // Only the upper 20 of the key's 30 bits are sorted (the lowest digit is
    // cleared, so the merges of larger clouds compare the same keys): 2^20
    // cells hold runs of 32 points about as compact as 2^30 for the clouds
    // sorted here, and one radix pass fewer is needed. The order only decides
    // which pairs the scans skip, never a result.
    uint32_t key[kSuper], val[kSuper];
#pragma unroll
    for (int u = 0; u < kSuper; ++u) {
        const int k = u * kSortT + tid;
        key[u] = 0;
        val[u] = (uint32_t)(c0 + k); // index within the sample
        if (k < n) {
            const float *p = pts + 3 * (size_t)k;
            key[u] =
                hilbert_key(quantize(p[0], f[0], scale), quantize(p[1], f[1], scale), quantize(p[2], f[2], scale)) &
                ~(uint32_t)(kBins - 1);
#pragma unroll
            for (int q = kFirstPass; q < kPasses; ++q)
                atomicAdd(&s.base[q - kFirstPass][(key[u] >> (q * kDigitBits)) & (kBins - 1)], 1);
        }
    }
    lds_barrier();
    // exclusive scans of the histograms: bin tid of every pass
#pragma unroll
    for (int q = kFirstPass; q < kPasses; ++q) {
        const int c = s.base[q - kFirstPass][tid];
        int inc = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(inc, o);
            if (lane >= o)
                inc += v;
        }
        if (lane == 63)
            s.wsum[wave] = inc;
        lds_barrier();
        int before = 0;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w)
            before += w < wave ? s.wsum[w] : 0;
        lds_barrier();
        s.base[q - kFirstPass][tid] = before + inc - c;
    }
    lds_barrier();
    static_assert(kPasses - kFirstPass == 2, "two passes, the keys in LDS between them");
    radix_pass(s, 1, n, key, val, [&](int pos, uint32_t k, uint32_t v) { s.mid[pos] = make_uint2(k, v); });
#pragma unroll
    for (int u = 0; u < kSuper; ++u) {
        const int k = u * kSortT + tid;
        const uint2 m = k < n ? s.mid[k] : make_uint2(0u, 0u);
        key[u] = m.x;
        val[u] = m.y;
    }
    radix_pass(s, 2, n, key, val, [&](int pos, uint32_t k, uint32_t v) {
        a.key[0][seg + pos] = k;
        a.val[0][seg + pos] = v;
    });
}

// Merges groups of `ways` sorted runs of `run` elements (the last ones
// shorter), one thread per element: its place in the group is its own index
// plus, for every other run, the elements there that come before it (an equal
// key of an earlier run does, so the order stays stable). K >= ways searches
// go side by side: what bounds this is the latency of a search's dependent
// loads, about log2(run), and for many points the loads themselves. 20000 +
// 20000 points: 8.4 us for the merge of ten chunks (34 us in two pairwise
// levels of serial merges); 4 x (65536 + 65536): 39 us in two levels of six
// (60 us in three pairwise ones, from four times larger chunks).
template <int K>
__global__ __launch_bounds__(kBlock) void k_sort_merge(SpatialArgs a, int run, int ways, int src)
{
    const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t nx = (int64_t)a.B * a.pad_x;
    const int cloud = g < nx ? 0 : 1;
    const int64_t h = cloud ? g - nx : g;
    const int pad = cloud ? a.pad_y : a.pad_x;
    if (h >= (int64_t)a.B * pad)
        return;
    const int b = (int)((uint32_t)h / (uint32_t)pad), k = (int)(h - (int64_t)b * pad); // h < 2^32
    const int n = cloud ? a.M : a.N;
    if (k >= n)
        return;
    const size_t seg = cloud ? nx + (size_t)b * pad : (size_t)b * pad;
    const uint32_t *sk = a.key[src] + seg;
    const uint32_t key = sk[k], val = a.val[src][seg + k];
    const int chunk = k / run, own = chunk % ways;
    const int p0 = (chunk - own) * run;
    int pos = k - own * run; // p0 + the index within the own run
    int lo[K], len[K], first[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
        const int64_t q = p0 + (int64_t)r * run;
        lo[r] = 0;
        len[r] = r < ways && r != own && q < n ? min(run, n - (int)q) : 0;
        first[r] = len[r] > 0 ? (int)q : k;
    }
    for (int step = 1 << (31 - __clz(run)); step > 0; step >>= 1) {
        uint32_t v[K];
#pragma unroll
        for (int r = 0; r < K; ++r) // in range also where lo + step is not
            v[r] = sk[first[r] + max(min(lo[r] + step, len[r]) - 1, 0)];
#pragma unroll
        for (int r = 0; r < K; ++r)
            lo[r] += ((lo[r] + step <= len[r]) & (v[r] < key + (r < own ? 1u : 0u))) ? step : 0; // keys are below 2^30
    }
#pragma unroll
    for (int r = 0; r < K; ++r)
        pos += lo[r];
    a.key[1 - src][seg + pos] = key;
    a.val[1 - src][seg + pos] = val;
}

__device__ __forceinline__ Box make_box(const float lo[3], const float hi[3])
{
    return Box{make_float4(lo[0], lo[1], lo[2], 0.0f), make_float4(hi[0], hi[1], hi[2], 0.0f)};
}

// The sorted points, the boxes of their runs and of the batch: one workgroup
// per (cloud, sample, batch of 64 runs).
__global__ __launch_bounds__(kSortT) void k_sort_gather(SpatialArgs a, int src)
{
    __shared__ float run_lo[64][3], run_hi[64][3];
    const int nbx = batches(a.pad_x), nby = batches(a.pad_y);
    const int cloud = blockIdx.x < (unsigned)a.B * nbx ? 0 : 1;
    const int h = cloud ? blockIdx.x - a.B * nbx : blockIdx.x;
    const int nbt = cloud ? nby : nbx, pad = cloud ? a.pad_y : a.pad_x;
    const int b = h / nbt, t = h - b * nbt;
    const int n = cloud ? a.M : a.N;
    const uint32_t *val = a.val[src] + (cloud ? (size_t)a.B * a.pad_x + (size_t)b * pad : (size_t)b * pad);
    const float *pts = (cloud ? a.y : a.x) + (size_t)b * n * 3;
#pragma unroll
    for (int u = 0; u < kSuper; ++u) {
        const int r = (u * kSortT + threadIdx.x) / kRun; // run within the batch
        const int k = t * kSortChunk + u * kSortT + threadIdx.x;
        float4 v = make_float4(0.0f, 0.0f, 0.0f, __int_as_float(-1));
        float lo[3] = {kInf, kInf, kInf}, hi[3] = {-kInf, -kInf, -kInf};
        if (k < n) {
            const uint32_t i = val[k];
            const float *p = pts + 3 * (size_t)i;
            v = make_float4(p[0], p[1], p[2], __uint_as_float(i));
            lo[0] = hi[0] = p[0];
            lo[1] = hi[1] = p[1];
            lo[2] = hi[2] = p[2];
        }
        if (k < pad)
            (cloud ? a.sy : a.sx)[(size_t)b * pad + k] = v;
        union_box<kRun>(lo, hi);
        if ((lane_id() & (kRun - 1)) == 0) {
            if (k < pad)
                (cloud ? a.box_y : a.box_x)[((size_t)b * pad + k) / kRun] = make_box(lo, hi);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                run_lo[r][c] = lo[c];
                run_hi[r][c] = hi[c];
            }
        }
    }
    lds_barrier();
    if (threadIdx.x >= 64)
        return;
    float lo[3], hi[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lo[c] = run_lo[threadIdx.x][c];
        hi[c] = run_hi[threadIdx.x][c];
    }
    union_box<64>(lo, hi);
    if (threadIdx.x == 0)
        (cloud ? a.batch_y : a.batch_x)[(size_t)b * nbt + t] = make_box(lo, hi);
}

// Box of each batch of 64 runs of the columns, with the runs' thresholds: one
// wave per (sample, batch), one lane per run (coalesced loads), then wave-wide
// min / max.
__global__ __launch_bounds__(kBlock) void k_batch_boxes(const Box *box, Box *batch, int B, int pad)
{
    const int64_t h = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int lane = lane_id();
    const int nbt = batches(pad);
    if (h >= (int64_t)B * nbt) // the whole wave
        return;
    const int b = (int)(h / nbt), t = (int)(h - (int64_t)b * nbt);
    const int runs = pad / kRun, r = t * 64 + lane;
    const Box *rb = box + (size_t)b * runs;
    float4 lo = make_float4(kInf, kInf, kInf, 0.0f), hi = make_float4(-kInf, -kInf, -kInf, -kInf);
    if (r < runs) {
        lo = rb[r].lo;
        hi = rb[r].hi;
    }
    for (int off = 32; off > 0; off >>= 1) {
        lo.x = fminf(lo.x, __shfl_xor(lo.x, off));
        lo.y = fminf(lo.y, __shfl_xor(lo.y, off));
        lo.z = fminf(lo.z, __shfl_xor(lo.z, off));
        hi.x = fmaxf(hi.x, __shfl_xor(hi.x, off));
        hi.y = fmaxf(hi.y, __shfl_xor(hi.y, off));
        hi.z = fmaxf(hi.z, __shfl_xor(hi.z, off));
        hi.w = fmaxf(hi.w, __shfl_xor(hi.w, off));
    }
    if (lane == 0)
        batch[(size_t)b * nbt + t] = Box{make_float4(lo.x, lo.y, lo.z, 0.0f), hi};
}

} // namespace

void launch_batch_boxes(const Box *box, Box *batch, int B, int pad, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_boxes, dim3(blocks_for(64 * (int64_t)B * batches(pad), kBlock)), dim3(kBlock), 0, s,
                       box, batch, B, pad);
}

hipError_t launch_spatial_sort(const SpatialArgs &a, hipStream_t s)
{
    const hipError_t e = set_dynamic_lds((const void *)k_spatial_sort, sizeof(SortLds));
    if (e != hipSuccess)
        return e;
    const int n_max = std::max(a.N, a.M);
    const int chunks = (n_max + kSortChunk - 1) / kSortChunk;
    hipLaunchKernelGGL(k_sort_frame, dim3(a.B * a.frame_slices), dim3(kSortT), 0, s, a);
    hipLaunchKernelGGL(k_spatial_sort, dim3(2 * a.B * chunks), dim3(kSortT), sizeof(SortLds), s, a);
    // as few levels as kMergeWays allows, each of as few runs as that takes
    int levels = 0, ways = 1;
    for (int64_t reach = 1; reach < chunks; reach *= kMergeWays)
        ++levels;
    for (int64_t reach = 0; levels > 0 && reach < chunks;) {
        ++ways;
        reach = 1;
        for (int l = 0; l < levels; ++l)
            reach *= ways;
    }
    const auto merge = ways <= 4    ? k_sort_merge<4>
                       : ways <= 6  ? k_sort_merge<6>
                       : ways <= 10 ? k_sort_merge<10>
                                    : k_sort_merge<kMergeWays>;
    int src = 0;
    int64_t run = kSortChunk;
    for (int l = 0; l < levels; ++l, run *= ways, src = 1 - src)
        hipLaunchKernelGGL(merge, dim3(blocks_for((int64_t)a.B * (a.pad_x + a.pad_y), kBlock)), dim3(kBlock), 0, s, a,
                           (int)std::min<int64_t>(run, n_max), ways, src);
    hipLaunchKernelGGL(k_sort_gather, dim3(a.B * (batches(a.pad_x) + batches(a.pad_y))), dim3(kSortT), 0, s, a, src);
    return hipGetLastError();
}

} // namespace apml
