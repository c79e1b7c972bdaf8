// N_D of the state vector on CDNA4 (gfx950): the number of dynamic objects
// in a frame, as the connected components of the pixels its custom stencil
// buffer marks (paper §III-D: the stencil buffer captures the dynamic
// objects, which are found by clustering it; Table IV: N_D; §IV-C, Eq. 1: an
// entry of E_t). A pixel is marked iff its stencil value is non-zero; two
// marked pixels are joined when they share an edge (4-connectivity) or an
// edge or a corner (8-connectivity).
//
// Pass 1, one workgroup per 64 x 32 tile: a thread loads eight adjacent pixels
// and turns them into bits, a row of the tile is a 64-bit mask, and each pixel's
// run of marked pixels, and where two rows touch, are bit operations. Union-find
// over the runs in LDS: a run's label sits at its first pixel, and links are
// made once per stretch where two rows touch, all rows at once (each thread
// those of its eight columns). Labels are in-tile indices; a union links the
// larger root under the smaller with an LDS atomicMin and retries from the old
// parent when another lane linked it first, so every label points to a smaller
// or equal index and every find ends. Only the labels that pass 2 can reach are
// stored, as frame-wide indices: those of the roots and of the marked pixels on
// the tile's edge. The tile adds its number of roots to the frame's count. A
// tile without marked pixels ends after its loads.
// Pass 2, two wavefronts per tile: its bottom row and right column are joined
// to their neighbours across the border with the same union-find in global
// memory (agent-scope atomics and loads), under the same rules for skipping
// implied links, and every link that joins two sets subtracts one from the
// count. The count is the number of sets left whatever the order of the links,
// so it is exact.
//
// Bound: latency (a byte per pixel is read; both passes are short dependent
// chains per tile). With 32 x 32 tiles, a label per pixel and the neighbours
// looked up in LDS, call time: 4 x 1440p without marked pixels 37 us, now 18; a
// 20 % / 60 % / 90 % random mask 354 / 574 / 488, now 255 / 285 / 229; fully
// marked 342, now 193; one 1080p frame with a rectangle 23, now 17. One
// wavefront per tile, without barriers, was slower where pixels are marked (46
// against 17 us on that frame: the rows' links one after the other); 512 threads
// of four columns each too, where the marked pixels form solid objects (4 x
// 1440p with rectangles 35.7 against 31.2 us). Those would suit one-pixel
// structures in small frames: one frame of 270 x 480 in one-pixel stripes takes
// 18.3 us, 14.4 with them and 14.2 before; a checkerboard 43, 26 and 39.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.h"

namespace exw {
namespace {

constexpr int kCcW = 64, kCcH = 32;             // tile (pixels)
constexpr int kCcThreads = kCcW * kCcH / 8;      // pass 1: eight adjacent pixels per thread
constexpr int kBorderTiles = 2;                  // pass 2: tiles per workgroup, two wavefronts each
constexpr int kBorderThreads = 128 * kBorderTiles;

__device__ __forceinline__ int lds_load(const int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ int lds_find(const int *lab, int x) {
    for (int p = lds_load(lab + x); p != x; p = lds_load(lab + x)) x = p;
    return x;
}

__device__ __forceinline__ void lds_union(int *lab, int a, int b) {
    for (;;) {
        a = lds_find(lab, a);
        b = lds_find(lab, b);
        if (a == b) return;
        const int hi = a > b ? a : b, lo = a > b ? b : a;
        const int old = atomicMin(lab + hi, lo);
        if (old == hi) return;  // hi was a root: linked
        a = old;                // hi had been linked meanwhile: join its parent too
        b = lo;
    }
}

__device__ __forceinline__ int g_load(const int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int g_find(const int *lab, int x) {
    for (int p = g_load(lab + x); p != x; p = g_load(lab + x)) x = p;
    return x;
}

// Returns the number of links that joined two sets (0 or 1).
__device__ __forceinline__ int g_union(int *lab, int a, int b) {
    for (;;) {
        a = g_find(lab, a);
        b = g_find(lab, b);
        if (a == b) return 0;
        const int hi = a > b ? a : b, lo = a > b ? b : a;
        const int old = __hip_atomic_fetch_min(lab + hi, lo, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
        if (old == hi) return 1;
        a = old;
        b = lo;
    }
}

struct CcArgs {
    const uint8_t *stencil;  // [N][H][W]
    int *labels;             // [N][H][W] frame-wide indices, of the roots and the tiles' edges
    uint32_t *count;         // [N], zero on entry to pass 1
    int h, w, tiles_x, tiles_per_frame, tiles;
    int first;               // tile of the launch's first workgroup
    int eight;               // 8-connectivity
};

__device__ __forceinline__ bool bit_at(uint64_t m, int i) { return (m >> i) & 1u; }

// First pixel of the run of marked pixels that pixel c of a row lies in.
__device__ __forceinline__ int run_start(uint64_t row, int c) {
    const uint64_t gaps = ~row & ((uint64_t(1) << c) - 1u);  // unmarked pixels left of c
    return gaps ? 64 - __clzll(static_cast<long long>(gaps)) : 0;
}

typedef uint64_t u64_u __attribute__((aligned(1)));

__global__ __launch_bounds__(kCcThreads) void cc_tile_kernel(CcArgs a) {
    __shared__ int lab[kCcW * kCcH];
    __shared__ uint64_t rows[kCcH + 1];  // marked pixels; a row past the last, empty
    __shared__ int roots[kCcThreads / 64];
    const int job = a.first + static_cast<int>(blockIdx.x);
    const int frame = job / a.tiles_per_frame;
    const int tile = job - frame * a.tiles_per_frame;
    const int x0 = (tile % a.tiles_x) * kCcW, y0 = (tile / a.tiles_x) * kCcH;
    const int64_t hw = static_cast<int64_t>(a.h) * a.w;
    const int r = threadIdx.x / 8, c0 = threadIdx.x % 8 * 8;  // row, first of eight columns
    // The thread's eight pixels as eight bits.
    uint32_t bits = 0;
    if (y0 + r < a.h) {
        const uint8_t *st = a.stencil + frame * hw + static_cast<int64_t>(y0 + r) * a.w + x0 + c0;
        if (x0 + c0 + 8 <= a.w) {
            uint64_t v = *reinterpret_cast<const u64_u *>(st);
            v |= v >> 4;
            v |= v >> 2;
            v |= v >> 1;
            // bit 0 of byte i to bit 56 + i (no two terms of the product meet)
            bits = static_cast<uint32_t>(((v & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56);
        } else {
            for (int i = 0; x0 + c0 + i < a.w && i < 8; ++i) bits |= (st[i] != 0 ? 1u : 0u) << i;
        }
    }
    reinterpret_cast<uint8_t *>(rows)[threadIdx.x] = static_cast<uint8_t>(bits);
    if (threadIdx.x == 0) rows[kCcH] = 0;
    if (!__syncthreads_or(bits != 0)) return;  // no marked pixel in the tile
    const uint64_t up = rows[r], dn = rows[r + 1];
    const uint64_t mine = uint64_t(0xff) << c0;
    // a run's label at its first pixel
    const uint64_t starts = up & ~(up << 1) & mine;
    for (uint64_t m = starts; m; m &= m - 1) {
        const int i = r * kCcW + __builtin_ctzll(m);
        lab[i] = i;
    }
    __syncthreads();
    // Links to the row below, made once per stretch where the two rows touch:
    // below at the stretch's first column (the pixel whose left and lower-left
    // neighbours are not both marked), a diagonal only where neither the pixel
    // beside nor the pixel below is marked.
    {
        const uint64_t both = up & dn;
        const uint64_t down = both & ~(both << 1);
        const uint64_t left = a.eight ? up & (dn << 1) & ~dn & ~(up << 1) : 0;
        const uint64_t right = a.eight ? up & (dn >> 1) & ~dn & ~(up >> 1) : 0;
        const int here = r * kCcW, below = here + kCcW;
        for (uint64_t m = down & mine; m; m &= m - 1) {
            const int c = __builtin_ctzll(m);
            lds_union(lab, here + run_start(up, c), below + run_start(dn, c));
        }
        for (uint64_t m = left & mine; m; m &= m - 1) {
            const int c = __builtin_ctzll(m);
            lds_union(lab, here + run_start(up, c), below + run_start(dn, c - 1));
        }
        for (uint64_t m = right & mine; m; m &= m - 1) {
            const int c = __builtin_ctzll(m);
            lds_union(lab, here + run_start(up, c), below + run_start(dn, c + 1));
        }
    }
    __syncthreads();
    int n_roots = 0;
    int *labels = a.labels + frame * hw;
    auto frame_index = [&](int i) { return (y0 + i / kCcW) * a.w + x0 + i % kCcW; };
    for (uint64_t m = starts; m; m &= m - 1) {
        const int i = r * kCcW + __builtin_ctzll(m);
        if (lds_load(lab + i) == i) {
            ++n_roots;
            labels[frame_index(i)] = frame_index(i);
        }
    }
    const uint64_t edge = r == 0 || r == kCcH - 1 ? up : up & ((uint64_t(1) << 63) | 1u);
    int last_start = -1, root = 0;  // neighbouring pixels of a run share its root
    for (uint64_t m = edge & mine; m; m &= m - 1) {
        const int c = __builtin_ctzll(m), s0 = run_start(up, c);
        if (s0 != last_start) root = frame_index(lds_find(lab, r * kCcW + s0));
        last_start = s0;
        labels[frame_index(r * kCcW + c)] = root;
    }
    // the tile's roots, one atomic per workgroup
    for (int off = 32; off > 0; off >>= 1) n_roots += __shfl_xor(n_roots, off);
    if (threadIdx.x % 64 == 0) roots[threadIdx.x / 64] = n_roots;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int k = 0; k < kCcThreads / 64; ++k) t += roots[k];
        atomicAdd(a.count + frame, static_cast<uint32_t>(t));
    }
}

// Two tiles per workgroup, two wavefronts per tile: the even one joins the
// tile's bottom row to the row below, the odd one its right column to the next.
__global__ __launch_bounds__(kBorderThreads) void cc_border_kernel(CcArgs a) {
    const int wave = static_cast<int>(threadIdx.x) / 64, lane = threadIdx.x % 64;
    const int job = a.first + static_cast<int>(blockIdx.x) * kBorderTiles + wave / 2;
    if (job >= a.tiles) return;
    const int frame = job / a.tiles_per_frame;
    const int tile = job - frame * a.tiles_per_frame;
    const int x0 = (tile % a.tiles_x) * kCcW, y0 = (tile / a.tiles_x) * kCcH;
    const int64_t hw = static_cast<int64_t>(a.h) * a.w;
    int *lab = a.labels + frame * hw;
    const uint8_t *st = a.stencil + frame * hw;
    // Whether a pixel is marked never changes: it is read from the stencil,
    // which the caches may serve (only the union-find needs coherent loads).
    // A lane's pixels are loaded before any is tested (clamped to the frame;
    // those outside it are unmarked).
    const bool bottom = wave % 2 == 0;  // wave-uniform
    // Bottom: lane l is column x0 + l of row y and of the row below; lanes 0
    // and 63 also load the columns beside the tile. Right: lane l is row
    // y0 - 1 + l of column x and of the next (lanes 1 .. 32 the tile's rows, 0
    // and 33 the rows beside it).
    const int x = bottom ? x0 + lane : x0 + kCcW - 1;
    const int y = bottom ? y0 + kCcH - 1 : y0 - 1 + min(lane, kCcH + 1);
    const int nx = bottom ? x : x + 1, ny = bottom ? y + 1 : y;  // across the border
    const int xe = lane == 0 ? x0 - 1 : x0 + kCcW;
    if ((bottom ? y : x) + 1 >= (bottom ? a.h : a.w)) return;  // wave-uniform: no neighbour
    const int px[4] = {x, nx, xe, xe}, py[4] = {y, ny, y, y + 1};
    uint8_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        v[k] = st[static_cast<int64_t>(min(max(py[k], 0), a.h - 1)) * a.w +
                  min(max(px[k], 0), a.w - 1)];
    bool mk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        mk[k] = px[k] >= 0 && px[k] < a.w && py[k] >= 0 && py[k] < a.h && v[k] != 0;
    const uint64_t mh = __ballot(mk[0]), mn = __ballot(mk[1]);  // here, across
    if (mh == 0) return;
    // The neighbours along the border, on this side and across it. Bottom row:
    // beyond lanes 0 and 63 the columns loaded beside the tile.
    const bool first = bottom ? lane == 0 : lane == 1;
    const bool mine = mk[0] && (bottom || (lane >= 1 && lane <= kCcH));
    const bool lf = lane > 0 ? bit_at(mh, lane - 1) : mk[2], ln = lane > 0 ? bit_at(mn, lane - 1) : mk[3];
    const bool rt = lane < 63 ? bit_at(mh, lane + 1) : mk[2], rn = lane < 63 ? bit_at(mn, lane + 1) : mk[3];
    int joined = 0;
    if (mine) {
        const int p = y * a.w + x, across = bottom ? p + a.w : p + 1, along = bottom ? 1 : a.w;
        // A link that the border's other links imply is skipped (the same
        // rules as inside the tiles, along the border).
        if (mk[1] && !(!first && lf && ln)) joined += g_union(lab, p, across);
        if (a.eight) {
            if (ln && !mk[1] && !lf) joined += g_union(lab, p, across - along);
            if (rn && !mk[1] && !rt) joined += g_union(lab, p, across + along);
        }
    }
    if (__ballot(joined != 0) == 0) return;  // wave-uniform
    for (int off = 32; off > 0; off >>= 1) joined += __shfl_xor(joined, off);
    if (lane == 0) atomicSub(a.count + frame, static_cast<uint32_t>(joined));
}

}  // namespace

size_t dynamic_objects_workspace_bytes(int n, int h, int w) {
    return sizeof(int) * static_cast<size_t>(n) * h * w;
}

hipError_t launch_dynamic_objects(const uint8_t *stencil, int n, int h, int w, int connectivity,
                                  uint32_t *count, void *workspace, hipStream_t stream) {
    hipError_t e = launch_zero_u32(count, n, stream);
    if (e != hipSuccess) return e;
    CcArgs a;
    a.stencil = stencil;
    a.labels = static_cast<int *>(workspace);
    a.count = count;
    a.h = h;
    a.w = w;
    a.tiles_x = (w + kCcW - 1) / kCcW;
    a.tiles_per_frame = a.tiles_x * ((h + kCcH - 1) / kCcH);
    a.eight = connectivity == 8;
    a.tiles = n * a.tiles_per_frame;  // below 2^31: the C ABI bounds the 32 x 32 tiles
    // One launch each, except for batches of millions of tiny frames (or frames
    // of a few columns and hundreds of millions of rows).
    auto launch = [&](auto kernel, int64_t threads, int tiles_each) {
        const int64_t group = kMaxWorkItems / threads * tiles_each;
        for (int64_t t0 = 0; t0 < a.tiles; t0 += group) {
            const int64_t some = a.tiles - t0 < group ? a.tiles - t0 : group;
            a.first = static_cast<int>(t0);
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((some + tiles_each - 1) / tiles_each)),
                               dim3(static_cast<unsigned>(threads)), 0, stream, a);
            if (e == hipSuccess) e = hipGetLastError();
        }
    };
    launch(cc_tile_kernel, kCcThreads, 1);
    if (e == hipSuccess) launch(cc_border_kernel, kBorderThreads, kBorderTiles);
    return e;
}

}  // namespace exw
