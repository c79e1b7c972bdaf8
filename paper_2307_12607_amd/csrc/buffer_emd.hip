// EMD features of the state vector on CDNA4 (gfx950): per frame and channel,
// the Earth Mover's Distance between the value distribution of a buffer of
// F_t and that of F_{t-1} (paper §III-D: the change of the world-normal and
// world-position buffers between frames is measured with the EMD; Table IV:
// EMD_{W_N}, EMD_{W_P}; §IV-C, Eq. 1: both are entries of E_t).
//
// Each channel's values are histogrammed over `bins` uniform bins on
// [lo, hi] (bin = floor((v - lo) * scale) in float64, clamped to the end
// bins; scale = bins / (hi - lo) from the host), and the one-dimensional EMD
// of the two unit-mass histograms is the L1 distance of their cumulative
// histograms times the bin width.
//
// Workgroups of 1024 threads (256 for many small planes) own a contiguous run
// of one plane of both buffers, count into LDS histograms (integer LDS atomics;
// both buffers' counts side by side) and add their non-zero bins to the plane's
// global counters with one integer atomic each. Smooth buffers put many lanes of a
// wavefront in one bin, and atomics on one address serialise: the workgroup
// keeps up to four copies of its histograms, lane l counting into copy l mod
// copies (the copies one word apart, so one bin of different copies falls in
// different banks), and adds the copies up at the end. Each lane takes 16
// consecutive bytes of each buffer at a time: one load where single values
// took four or eight, and neighbouring pixels, which tend to share a bin, in
// one lane, which adds a run of them at once. The last workgroup of a plane (by
// a ticket; the only one takes its LDS histograms as they are) scans the count
// differences in 64-bit integers and sums their magnitudes exactly; the result
// is that exact sum / (H*W) * width in float64. Integer counts make every result
// independent of the order of the atomics.
//
// Bound: the LDS additions and the float64 binning (six operations per value),
// with HBM close behind (4.4 TB/s on f32). Before (256 threads, single-value
// loads, a floor and two float64 clamps per value, one addition per value, the
// sums in a launch of their own), call time: three channels of 4 x 1440p f32,
// 1024 bins 104 us on smooth, 96 on random and 100 on equal values, now 82, 81
// and 81 (93, 83 and 99 with one addition per value); bf16, 256 bins 88, 54 and
// 84, now 46, 46 and 44 (80, 43 and 84); one 1080p frame f32 28, now 25; 2 x 481
// x 270 19.9, now 16.3.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.h"
#include "warp_common.h"

namespace exw {
namespace {

constexpr int kEmdSlots = 512;                         // workgroups of 1024 the chip holds: two per CU
constexpr int64_t kEmdRun = 8192;                      // values of a plane per workgroup, at least
constexpr int64_t kEmdMerge = 128 * 1024;              // see emd_plan

constexpr int kEmdLdsWords = 8200;                     // LDS words for the copies, at most (~32 KB)

struct EmdArgs {
    const void *cur, *prev;
    int64_t hw;
    int parts;
    int64_t run;       // values per workgroup (the last one may hold fewer)
    double lo, scale;  // bin = floor((v - lo) * scale), clamped
    int bins;
    int copies;        // LDS copies of the two histograms (1, 2 or 4)
    int stride;        // words from one copy to the next: 2 * bins + 1
    uint32_t *counts;  // [planes][2][bins], zero on entry
    double width;      // of a bin
    double *emd;       // [planes]; the first word of each is the ticket, zero on entry
};

// floor((v - lo) * scale) clamped to [0, bins - 1], NaN to 0: the conversion
// truncates and saturates, and takes NaN to 0 (a truncated value differs from
// the floor only below 0, where both are clamped).
__device__ __forceinline__ int bin_of(float v, double lo, double scale, int bins) {
    const double t = (static_cast<double>(v) - lo) * scale;
    int i;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(t));
    return min(max(i, 0), bins - 1);
}


__device__ __forceinline__ long long wave_sum_i64(long long v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
    return v;
}

// S = sum_i |CA_i - CB_i| over the cumulative counts of one plane, in 64-bit
// integers (exact), then S / (H*W) * width; by the whole workgroup. diff(i):
// the difference of the two buffers' counts of bin i.
template <int NT, typename Diff>
__device__ __forceinline__ void emd_of_plane(const EmdArgs &a, int plane, long long *lds,
                                             Diff &&diff) {
    constexpr int kWaves = NT / 64;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int per = (a.bins + NT - 1) / NT;
    const int b0 = min(a.bins, static_cast<int>(threadIdx.x) * per);
    const int b1 = min(a.bins, b0 + per);
    long long run = 0;
    for (int i = b0; i < b1; ++i) run += diff(i);
    // exclusive scan of the threads' totals: within the wavefront, then over
    // the wavefronts' totals
    long long inc = run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const long long up = __shfl_up(inc, d);
        if (lane >= d) inc += up;
    }
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    long long cum = inc - run;  // differences of the bins before b0
    for (int k = 0; k < wave; ++k) cum += lds[k];
    long long s = 0;
    for (int i = b0; i < b1; ++i) {
        cum += diff(i);
        s += cum < 0 ? -cum : cum;
    }
    s = wave_sum_i64(s);
    if (lane == 0) lds[kWaves + wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int k = 0; k < kWaves; ++k) t += lds[kWaves + k];
        a.emd[plane] = static_cast<double>(t) / static_cast<double>(a.hw) * a.width;
    }
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void emd_kernel(EmdArgs a) {
    extern __shared__ uint32_t lds[];  // [copies][stride]: [2][bins] and a pad word each
    __shared__ long long scan[2 * (NT / 64)];
    __shared__ int last;
    constexpr int V = 16 / sizeof(T);  // values per load
    // (element-aligned: planes of odd size put them at any multiple of it)
    typedef T vec __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    const int plane = static_cast<int>(blockIdx.x) / a.parts;
    const int part = static_cast<int>(blockIdx.x) - plane * a.parts;
    for (int i = threadIdx.x; i < a.copies * a.stride; i += NT) lds[i] = 0u;
    __syncthreads();
    uint32_t *hist = lds + (static_cast<int>(threadIdx.x) & (a.copies - 1)) * a.stride;
    const T *pa = static_cast<const T *>(a.cur) + static_cast<int64_t>(plane) * a.hw;
    const T *pb = static_cast<const T *>(a.prev) + static_cast<int64_t>(plane) * a.hw;
    const int64_t begin = static_cast<int64_t>(part) * a.run;
    const int64_t end = min(a.hw, begin + a.run);
    auto bin = [&](T v) { return bin_of(to_f32(v), a.lo, a.scale, a.bins); };
    // V neighbouring values: one addition per run of values of one bin.
    auto count = [&](const vec &v, uint32_t *to) {
        int run_bin = bin(v[0]);
        uint32_t run = 1u;
#pragma unroll
        for (int q = 1; q < V; ++q) {
            const int b = bin(v[q]);
            if (b != run_bin) {
                atomicAdd(&to[run_bin], run);
                run = 0u;
                run_bin = b;
            }
            ++run;
        }
        atomicAdd(&to[run_bin], run);
    };
    const int64_t whole = begin + (end - begin) / V * V;  // full loads end here
    int64_t i = begin + static_cast<int64_t>(threadIdx.x) * V;
    constexpr int64_t kStep = static_cast<int64_t>(NT) * V;
    if (i < whole) {
        vec na = *reinterpret_cast<const vec *>(pa + i), nb = *reinterpret_cast<const vec *>(pb + i);
        for (; i < whole; i += kStep) {
            const vec va = na, vb = nb;
            const int64_t j = i + kStep < whole ? i + kStep : i;  // (the next load is in flight)
            na = *reinterpret_cast<const vec *>(pa + j);
            nb = *reinterpret_cast<const vec *>(pb + j);
            count(va, hist);
            count(vb, hist + a.bins);
        }
    }
    if (const int64_t t = whole + threadIdx.x; t < end) {
        atomicAdd(&hist[bin(pa[t])], 1u);
        atomicAdd(&hist[a.bins + bin(pb[t])], 1u);
    }
    __syncthreads();
    auto total = [&](int k) {  // count k over the copies
        uint32_t t = lds[k];
        for (int c = 1; c < a.copies; ++c) t += lds[c * a.stride + k];
        return t;
    };
    if (a.parts == 1) {  // every count of the plane is here
        emd_of_plane<NT>(a, plane, scan, [&](int i) {
            return static_cast<long long>(total(i)) - total(a.bins + i);
        });
        return;
    }
    uint32_t *g = a.counts + static_cast<int64_t>(plane) * 2 * a.bins;
    for (int k = threadIdx.x; k < 2 * a.bins; k += NT)
        if (const uint32_t t = total(k); t != 0u) atomicAdd(&g[k], t);
    // Every addition of this workgroup has been made (they are device-wide
    // atomics, read back as such) before the ticket says so. One thread's fence
    // per workgroup: one per thread wrote the L2 back 1024 times (145 against
    // 22 us).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(reinterpret_cast<unsigned *>(a.emd + plane), 1u) ==
               static_cast<unsigned>(a.parts) - 1u;
    }
    __syncthreads();
    if (!last) return;
    auto count_of = [&](int k) -> long long {  // after the other workgroups' adds
        return __hip_atomic_load(g + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    emd_of_plane<NT>(a, plane, scan, [&](int i) { return count_of(i) - count_of(a.bins + i); });
}

// The counters and the tickets (the first word of every result).
__global__ __launch_bounds__(256) void emd_zero_kernel(uint32_t *counts, int64_t n, double *emd,
                                                       int64_t planes) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    for (int64_t i = t; i < n; i += stride) counts[i] = 0u;
    for (int64_t i = t; i < planes; i += stride) emd[i] = 0.0;
}

// Workgroups per plane and their size.
struct EmdPlan {
    int parts, threads;
};

// Workgroups of 1024 work in rounds of kEmdSlots; a round takes the time of its
// runs plus, where a plane has several workgroups, what it takes to merge and
// hand over their counts, about that of kEmdMerge bytes of each buffer (17 to 21
// us for 256 and 1024 bins). The parts that give the least of it, at runs of
// kEmdRun values at least: as many as one round holds while there are few
// planes (24 planes of 1440p: 21), one from a few hundred small planes on (900
// planes of 480 x 270 f32, 1024 bins: 166 us, two parts 257, four 338), and a few
// parts where that fills the last round (258 planes of 1080p bf16, 256 bins:
// one part 662 us, two 529, three 483, five 467, nine 484, twenty 598).
// Workgroups of 256 where the planes are small and many: there the clearing,
// the barriers and the scan of the bins count (6000 planes of 64 x 64 f32, 256
// bins: 34 us, 62 with 1024; 20000 of 16 x 16, 64 bins: 40 and 163). Many bins
// keep the larger ones (6000 of 32 x 32, 4096 bins: 72 us, 100 with 256).
EmdPlan emd_plan(int64_t planes, int64_t hw, int esize, int bins) {
    const int64_t want = (hw + kEmdRun - 1) / kEmdRun;
    auto rounds_time = [&](int64_t parts) {
        const int64_t rounds = (planes * parts + kEmdSlots - 1) / kEmdSlots;
        return rounds * (hw * esize / parts + (parts > 1 ? kEmdMerge : 0));
    };
    int64_t parts = 1, best = rounds_time(1);
    const int64_t first = planes < kEmdSlots ? kEmdSlots / planes : 1;  // one round full
    for (int64_t p = first < want ? first : want; p <= want && p <= first + 8; ++p)
        if (const int64_t t = rounds_time(p); t < best) { parts = p; best = t; }
    const bool small = planes > kEmdSlots && hw <= 32768 && bins <= 512;
    return EmdPlan{static_cast<int>(parts), parts == 1 && small ? 256 : 1024};
}

template <typename T>
void launch_hist(int threads, dim3 grid, const EmdArgs &a, hipStream_t st) {
    const size_t lds = sizeof(uint32_t) * a.copies * a.stride;
    if (threads == 256)
        hipLaunchKernelGGL((emd_kernel<T, 256>), grid, dim3(256), lds, st, a);
    else
        hipLaunchKernelGGL((emd_kernel<T, 1024>), grid, dim3(1024), lds, st, a);
}

}  // namespace

size_t buffer_emd_workspace_bytes(int n, int c, int bins) {
    return sizeof(uint32_t) * 2 * static_cast<size_t>(n) * c * bins;
}

hipError_t launch_buffer_emd(int dtype, const void *cur, const void *prev, int n, int c, int h,
                             int w, double lo, double hi, int bins, double *emd, void *workspace,
                             hipStream_t stream) {
    const int64_t planes = static_cast<int64_t>(n) * c;
    uint32_t *counts = static_cast<uint32_t *>(workspace);
    EmdArgs a;
    a.hw = static_cast<int64_t>(h) * w;
    a.stride = 2 * bins + 1;
    a.copies = 4;
    while (a.copies > 1 && a.copies * a.stride > kEmdLdsWords) a.copies /= 2;
    const EmdPlan plan = emd_plan(planes, a.hw, dtype == 0 ? 4 : 2, bins);
    a.parts = plan.parts;
    a.run = ((a.hw + a.parts - 1) / a.parts + 7) / 8 * 8;  // a multiple of 16 bytes
    a.parts = static_cast<int>((a.hw + a.run - 1) / a.run);
    a.width = (hi - lo) / static_cast<double>(bins);
    a.lo = lo;
    a.scale = static_cast<double>(bins) / (hi - lo);
    a.bins = bins;
    hipError_t e = hipSuccess;
    if (a.parts > 1) {
        const int64_t words = planes * 2 * bins;
        const int64_t blocks = (words + 255) / 256 < 1024 ? (words + 255) / 256 : 1024;
        hipLaunchKernelGGL(emd_zero_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                           stream, counts, words, emd, planes);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // One launch, except for batches of millions of tiny planes (a plane has at
    // most kEmdSlots + 8 workgroups, so any plane fits a launch).
    const int64_t group = kMaxWorkItems / plan.threads / a.parts;
    const int64_t plane_bytes = a.hw * (dtype == 0 ? 4 : 2);
    for (int64_t p0 = 0; p0 < planes; p0 += group) {
        const int64_t some = planes - p0 < group ? planes - p0 : group;
        const dim3 grid(static_cast<unsigned>(some * a.parts));
        a.cur = static_cast<const char *>(cur) + p0 * plane_bytes;
        a.prev = static_cast<const char *>(prev) + p0 * plane_bytes;
        a.counts = counts + p0 * 2 * bins;
        a.emd = emd + p0;
        switch (dtype) {
        case 0: launch_hist<float>(plan.threads, grid, a, stream); break;
        case 1: launch_hist<_Float16>(plan.threads, grid, a, stream); break;
        default: launch_hist<__bf16>(plan.threads, grid, a, stream); break;
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace exw
