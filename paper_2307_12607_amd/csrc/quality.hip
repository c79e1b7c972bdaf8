// Frame quality on CDNA4 (gfx950): per-frame MSE, PSNR and SSIM of a
// predicted frame against the ground truth (paper §IV-C1: the decision
// predictor's reward is the gain in PSNR = 10 log10(peak^2 / MSE) and in
// SSIM of the chosen action's frame over the other action's frame).
//
// SSIM is the Gaussian-window index (11 x 11 window, standard deviation 1.5,
// C1 = (0.01 peak)^2, C2 = (0.03 peak)^2) evaluated where the window lies
// inside the frame and averaged over those positions and the channels. The
// index needs four window sums: of x, y, x^2 + y^2 (only the sum of the two
// variances enters) and x y. The window is separable. A workgroup of NW
// wavefronts owns a strip of 64 NW input columns of one channel, a column per
// lane, and walks down its rows: each row's four values are added into the
// eleven output rows they feed, held in float64 registers as a ring of twelve
// slots (indexed at compile time: batches of four rows, unrolled by three).
// Four finished rows at a time go through LDS, where each lane takes four
// adjacent output columns of one row: 14 columns are read for 4 outputs, so
// LDS moves 14 / 4 values per output and sum instead of 11. The squared errors
// for the MSE are summed on the way. Partials are folded per frame in an
// order fixed by the batch's shape, so the results are reproducible bit for bit.
//
// Bound: the float64 vector ALU, which issues at the rate of unpacked float32
// (float32 sums would lose the low digits of E[x^2] - E[x]^2). Operations per
// output: 44 fused multiply-adds vertically, 44 horizontally, ~12 to form the
// four values and convert, ~30 for the index. Filtering horizontally first,
// each lane its own column from LDS (22 reads, 22 conversions, 7 operations per
// tap for five sums) took ~190 and 15 % more for the halo rows:
// 24 x 1080p RGBA f32 1500 us before, 1034 us now.
#include <cmath>

#include "launch.h"
#include "warp_common.h"

namespace exw {
namespace {

constexpr int kWin = 11;
constexpr int kHalo = kWin - 1;
constexpr int kBatch = 4;  // rows of window sums that go through LDS together
constexpr int kRing = 12;  // accumulating output rows: a multiple of kBatch, at least kWin

// The partials' room in the caller's workspace: one per strip of 64 x 66
// outputs, which the strips of a launch never outnumber.
constexpr int kRoomW = 64, kRoomRows = 66;

struct QualityArgs {
    const void *pred, *truth;
    int h, w;
    int strips_x, strips_y;
    int strip_rows;   // output rows of a strip
    double g[kWin];  // normalised 1-D Gaussian weights
    double c1, c2;
    double *partial;  // [B][C][strips_y][strips_x][2] = (ssim sum, squared-error sum)
};

typedef double f64x2 __attribute__((ext_vector_type(2)));

template <typename T, int NW>
__global__ __launch_bounds__(64 * NW, 2) void ssim_strip_kernel(QualityArgs a) {
    constexpr int kCols = 64 * NW;           // input columns of a strip
    constexpr int kOut = kCols - kHalo;      // output columns
    constexpr int kGroups = kCols / 4;       // groups of four adjacent columns
    // Window sums of kBatch rows after the vertical filter. Four columns take
    // six doubles: lanes then read their groups, 48 bytes apart, without bank
    // conflicts. (One group more than written: read by the last groups, whose
    // outputs past kOut are dropped.)
    __shared__ __attribute__((aligned(16))) double vsum[kBatch][4][(kGroups + 1) * 6];
    __shared__ double red[2][NW];
    const int tid = threadIdx.x;
    int blk = blockIdx.x;
    const int sx = blk % a.strips_x;
    blk /= a.strips_x;
    const int sy = blk % a.strips_y;
    const int pl = blk / a.strips_y;  // channel plane: frame * C + channel
    const int w = a.w, h = a.h;
    const int64_t plane = pl * (static_cast<int64_t>(h) * w);
    const int j0 = sx * kOut, i0 = sy * a.strip_rows;
    const T *px = static_cast<const T *>(a.pred) + plane + min(j0 + tid, w - 1);
    const T *py = static_cast<const T *>(a.truth) + plane + min(j0 + tid, w - 1);
    const bool last_x = sx == a.strips_x - 1, last_y = sy == a.strips_y - 1;
    // Input rows this strip reads, and the pixels whose squared errors it owns.
    const int rows_out = min(a.strip_rows, h - kHalo - i0);
    const int rows_in = rows_out + kHalo;
    const int own_rows = last_y ? h - i0 : a.strip_rows;
    const bool own_col = j0 + tid < w && (last_x || tid < kOut);
    // This lane's outputs in the horizontal filter.
    const int grp = tid % kGroups, grow = tid / kGroups;
    const int cols_out = min(kOut, w - kHalo - j0) - 4 * grp;  // of its four columns

    double acc[kRing][4];
#pragma unroll
    for (int s = 0; s < kRing; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[s][q] = 0.0;
    double ssim_sum = 0.0, sq_sum = 0.0;

    // The next batch of rows is loaded while the current one is filtered (rows
    // past the strip repeat its last: what they add to is never output).
    T nx[kBatch], ny[kBatch];
    auto load = [&](int r0) {
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const int64_t row = static_cast<int64_t>(i0 + min(r0 + q, rows_in - 1)) * w;
            nx[q] = px[row];
            ny[q] = py[row];
        }
    };
    load(0);
    for (int base = 0; base < rows_in; base += kRing) {
#pragma unroll
        for (int bt = 0; bt < kRing / kBatch; ++bt) {
            const int r0 = base + bt * kBatch;  // first input row of the batch
            if (r0 >= rows_in) break;           // workgroup-uniform
            T cx[kBatch], cy[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) { cx[q] = nx[q]; cy[q] = ny[q]; }
            load(r0 + kBatch);
            double batch_sq = 0.0;  // (fewer additions to the long sum)
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int s = bt * kBatch + q;
                const double x = to_f32(cx[q]), y = to_f32(cy[q]);
                if (r0 + q < own_rows && own_col) {
                    const double d = x - y;
                    batch_sq = fma(d, d, batch_sq);
                }
                const double v[4] = {x, y, fma(x, x, y * y), x * y};
                // input row r feeds output rows r - t, t = 0 .. 10, kept in
                // ring slot (r - t) mod 12 = (s - t) mod 12 (static)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    acc[s][k] = a.g[0] * v[k];
#pragma unroll
                    for (int t = 1; t < kWin; ++t) {
                        const int slot = (s - t + kRing) % kRing;
                        acc[slot][k] = fma(a.g[t], v[k], acc[slot][k]);
                    }
                    // output row r - 10 is complete
                    vsum[q][k][tid + 2 * (tid / 4)] = acc[(s + kRing - kHalo) % kRing][k];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            sq_sum += batch_sq;
            __syncthreads();
            const int r_out = r0 + grow - kHalo;  // this lane's output row
            if (r_out >= 0 && r_out < rows_out && cols_out > 0) {
                double o[4][4];  // [sum][column]
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const f64x2 *src = reinterpret_cast<const f64x2 *>(&vsum[grow][k][grp * 6]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[k][j] = 0.0;
#pragma unroll
                    for (int m = 0; m < 7; ++m) {  // columns 2 m, 2 m + 1 of the 14
                        const f64x2 p = src[(m / 2) * 3 + m % 2];
#pragma unroll
                        for (int e = 0; e < 2; ++e)
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const int b = 2 * m + e - j;
                                if (b >= 0 && b < kWin) o[k][j] = fma(a.g[b], e ? p.y : p.x, o[k][j]);
                            }
                    }
                    __builtin_amdgcn_sched_barrier(0);  // one sum's columns in registers at a time
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double mx = o[0][j], my = o[1][j];
                    const double mxy = mx * my, mm = fma(mx, mx, my * my);
                    const double num = fma(2.0, mxy, a.c1) * fma(2.0, o[3][j] - mxy, a.c2);
                    const double den = (mm + a.c1) * ((o[2][j] - mm) + a.c2);
                    if (j < cols_out) ssim_sum += num / den;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __syncthreads();  // the sums have been read
        }
    }
    // wavefront sums (butterfly; addition is commutative, so every lane
    // agrees), then the wavefronts in order
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        ssim_sum += __shfl_xor(ssim_sum, m);
        sq_sum += __shfl_xor(sq_sum, m);
    }
    if (tid % 64 == 0) {
        red[0][tid / 64] = ssim_sum;
        red[1][tid / 64] = sq_sum;
    }
    __syncthreads();
    if (tid < 2) {
        double t = red[tid][0];
        for (int k = 1; k < NW; ++k) t += red[tid][k];
        const int64_t idx = (static_cast<int64_t>(pl) * a.strips_y + sy) * a.strips_x + sx;
        a.partial[2 * idx + tid] = t;
    }
}

// One wavefront per frame folds its partials in a fixed order.
__global__ __launch_bounds__(64) void quality_final_kernel(const double *partial, int per_frame,
                                                           double n_px, double n_pos,
                                                           double peak, double *quality) {
    const int frame = blockIdx.x;
    const double *p = partial + 2 * static_cast<int64_t>(frame) * per_frame;
    double s = 0.0, q = 0.0;
    for (int i = threadIdx.x; i < per_frame; i += 64) {
        s += p[2 * i];
        q += p[2 * i + 1];
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        s += __shfl_xor(s, m);
        q += __shfl_xor(q, m);
    }
    if (threadIdx.x == 0) {
        const double mse = q / n_px;
        quality[3 * frame] = mse;
        quality[3 * frame + 1] = 10.0 * log10(peak * peak / mse);
        quality[3 * frame + 2] = s / n_pos;
    }
}

// Strips of the workspace's room per channel.
void room(int h, int w, int &sx, int &sy) {
    sx = (w - kHalo + kRoomW - 1) / kRoomW;
    sy = (h - kHalo + kRoomRows - 1) / kRoomRows;
}

// Wavefronts per strip, strips across a plane and output rows of a strip.
struct StripPlan {
    int nw, strips_x, rows;
};

// The plan of least estimated time, in units of one operation of a wavefront:
// a wavefront filters its rows and the halo's vertically (92 per row), its
// output rows horizontally with the index (111), and pays about 600 once. The
// chip holds 2048 of these wavefronts, two per SIMD, in a round; fewer than half
// of that (one per SIMD) take 0.6 of a round, and after full rounds 0.35 to 0.5
// (measured; strips of two wavefronts then pair up on half of the SIMDs). So:
// the fewest wavefronts that cover the width with strips of 54, 118 or 246
// outputs (776 planes of 150 x 257: five of one wavefront 184 us, two of four
// took 516), strips of even height (150 rows as 70 and 70 outputs, not 132 and
// 8), and short ones where there are few planes (one 1080p RGBA frame: 16 strips
// of 67 rows 53 us, 45 of 24 took 68). At most 136 rows where the room allows
// (a lane's sums stay short), and no more strips than the workspace's room.
// Widths of 65 to 74 columns pay two wavefronts where filtering horizontally
// first took one, ten of whose lanes loaded twice: 3076 planes of 150 x 65
// 285 us against 245.
StripPlan strip_plan(int64_t planes, int h, int w) {
    constexpr int64_t kSlots = 2048;
    const int out_w = w - kHalo, out_h = h - kHalo;
    int room_x, room_y;
    room(h, w, room_x, room_y);
    StripPlan best{4, 0, 0};
    double best_time = 0.0;
    int64_t best_waves = 0;
    for (int nw = 4; nw >= 1; nw /= 2) {
        const int sx = (out_w + 64 * nw - kHalo - 1) / (64 * nw - kHalo);
        const int64_t fit = static_cast<int64_t>(room_x) * room_y / sx;
        if (fit < 1) continue;  // (four wavefronts always fit: sx <= room_x)
        int64_t least = (out_h + 135) / 136, most = (out_h + 7) / 8;
        if (most > 64 + least) most = 64 + least;
        if (most > fit) most = fit;
        if (least > most) least = most;
        for (int64_t n = least; n <= most; ++n) {
            const int rows = static_cast<int>((out_h + n - 1) / n);
            const int64_t waves = planes * sx * nw * ((out_h + rows - 1) / rows);
            const int64_t full = waves / kSlots, rest = waves % kSlots;
            double part = rest == 0 ? 0.0 : 1.0;
            if (rest > 0 && rest <= kSlots / 2) {
                part = 0.6;
                if (full > 0) part = rest <= kSlots / 4 ? 0.35 : (nw == 2 ? 0.85 : 0.5);
            }
            const double time = (static_cast<double>(full) + part) *
                                ((rows + kHalo + 3) / 4 * 4 * 92.0 + rows * 111.0 + 600.0);
            if (best.rows == 0 || time < best_time || (time == best_time && waves < best_waves)) {
                best = StripPlan{nw, sx, rows};
                best_time = time;
                best_waves = waves;
            }
            if (waves > 8 * kSlots) break;  // shorter strips only add halo rows
        }
    }
    return best;
}

template <typename T>
void launch_strips(int nw, dim3 grid, hipStream_t st, const QualityArgs &a) {
    switch (nw) {
    case 1: hipLaunchKernelGGL((ssim_strip_kernel<T, 1>), grid, dim3(64), 0, st, a); break;
    case 2: hipLaunchKernelGGL((ssim_strip_kernel<T, 2>), grid, dim3(128), 0, st, a); break;
    default: hipLaunchKernelGGL((ssim_strip_kernel<T, 4>), grid, dim3(256), 0, st, a); break;
    }
}

}  // namespace

size_t quality_workspace_bytes(int b, int c, int h, int w) {
    int sx, sy;
    room(h, w, sx, sy);
    return sizeof(double) * 2 * static_cast<size_t>(b) * c * sx * sy;
}

hipError_t launch_quality(int dtype, const void *pred, const void *truth, int b, int c, int h,
                          int w, double peak, double *quality, void *workspace,
                          hipStream_t stream) {
    QualityArgs a;
    a.h = h;
    a.w = w;
    const StripPlan plan = strip_plan(static_cast<int64_t>(b) * c, h, w);
    const int nw = plan.nw;
    a.strips_x = plan.strips_x;
    a.strip_rows = plan.rows;
    a.strips_y = (h - kHalo + plan.rows - 1) / plan.rows;
    double e[kWin], sum = 0.0;
    for (int i = 0; i < kWin; ++i) {
        const double r = i - (kWin - 1) / 2;
        e[i] = std::exp(-(r * r) / (2.0 * 1.5 * 1.5));
        sum += e[i];
    }
    for (int i = 0; i < kWin; ++i) a.g[i] = e[i] / sum;
    a.c1 = (0.01 * peak) * (0.01 * peak);
    a.c2 = (0.03 * peak) * (0.03 * peak);
    double *partial = static_cast<double *>(workspace);
    const int64_t planes = static_cast<int64_t>(b) * c;
    const int64_t per_plane = static_cast<int64_t>(a.strips_x) * a.strips_y;
    // One launch, except for batches whose strips would exceed it (tens of
    // millions of tiny planes).
    const int64_t fit = kMaxWorkItems / (64 * nw) / per_plane;
    const int64_t group = fit < 1 ? 1 : fit;
    const int64_t plane_bytes = static_cast<int64_t>(h) * w * (dtype == 0 ? 4 : 2);
    for (int64_t p0 = 0; p0 < planes; p0 += group) {
        const int64_t some = planes - p0 < group ? planes - p0 : group;
        const dim3 grid(static_cast<unsigned>(some * per_plane));
        a.pred = static_cast<const char *>(pred) + p0 * plane_bytes;
        a.truth = static_cast<const char *>(truth) + p0 * plane_bytes;
        a.partial = partial + 2 * p0 * per_plane;
        switch (dtype) {
        case 0: launch_strips<float>(nw, grid, stream, a); break;
        case 1: launch_strips<_Float16>(nw, grid, stream, a); break;
        default: launch_strips<__bf16>(nw, grid, stream, a); break;
        }
        if (const hipError_t err = hipGetLastError(); err != hipSuccess) return err;
    }
    const double n_px = static_cast<double>(c) * h * w;
    const double n_pos = static_cast<double>(c) * (h - kHalo) * (w - kHalo);
    hipLaunchKernelGGL(quality_final_kernel, dim3(static_cast<unsigned>(b)), dim3(64), 0, stream,
                       partial, static_cast<int>(c * per_plane), n_px, n_pos, peak, quality);
    return hipGetLastError();
}

}  // namespace exw
