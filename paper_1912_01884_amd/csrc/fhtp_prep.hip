// Optional input steps before the band FHT: the transpose that turns mostly
// horizontal curves into mostly vertical ones (Fig. 7), and the row-wise
// smoothing of the main problem's step 1.
//
// Smoothing reads the Gaussian of step 1 as the binomial kernel C(2r, i),
// i = 0 .. 2r (variance r/2), with each row extended by repeating its end
// pixels and the sum normalised by 4^r with rounding half up, so the whole
// path stays exact integer arithmetic and the result keeps the pixel type.
//
// One workgroup makes a 64 x 64 tile of the detection image.  It stages the
// source rows of the tile plus an r-column halo in LDS, reading the input
// along its own rows (so the transposed case reads coalesced too, a wave one
// row of 64 pixels a load, every load of the tile in flight at once), then each
// thread makes four adjacent outputs of a row from 4 + 2r staged pixels and
// stores them together where the output's alignment allows.  The radius is a
// template constant: the taps are constants and nothing is divided.
//
// What bounds it: the image read and written once, 16.8 MB at 2048 x 2048, 16-bit
// pixels, radius 2, transposed: 8.0 us a launch in a detection (events), 17.9
// with a division per staged pixel, run-time taps and one output per store.
#include "fhtp_internal.h"

namespace fhtp {
namespace {

constexpr int kTile = 64;
constexpr int kMaxRadius = 7;
constexpr int kThreads = 256;

struct PrepArgs {
    const void* img;
    void* out;
    int ws;      // input columns
    int ho, wo;  // detection image dimensions
    int vec;     // four outputs at a multiple of four columns are one aligned store
};

// C(2r, i)
constexpr int binomial(int n, int i) {
    int c = 1;
    for (int q = 1; q <= i; ++q) c = c * (n - q + 1) / q;
    return c;
}

template <typename PixT, int R, bool TRANSPOSE>
__global__ __launch_bounds__(kThreads) void prep_kernel(PrepArgs a) {
    constexpr int kSpan = kTile + 2 * R;   // staged columns
    constexpr int kPitch = kSpan | 1;      // odd: no bank conflicts either way
    constexpr int kWaves = kThreads / 64;
    __shared__ int tile[kTile * kPitch];
    const PixT* __restrict__ img = static_cast<const PixT*>(a.img);
    PixT* __restrict__ out = static_cast<PixT*>(a.out);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x0 = blockIdx.x * kTile;  // detection columns of the tile
    for (int y0 = blockIdx.y * kTile; y0 < a.ho; y0 += gridDim.y * kTile) {
        // Stage S(y, x) for y in [y0, y0 + 64), x in [x0 - R, x0 + 64 + R); x and,
        // past the image's last row, y clamped (the latter's outputs are not stored).
        if constexpr (!TRANSPOSE) {
            constexpr int kRows = kTile / kWaves;  // rows of a wave
            const int xa = min(max(x0 - R + lane, 0), a.wo - 1);
            const int xb = min(x0 - R + 64 + lane, a.wo - 1);
            PixT p[kRows], q[R > 0 ? kRows : 1];
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                const PixT* row = img + (size_t)min(y0 + wave + i * kWaves, a.ho - 1) * a.ws;
                p[i] = row[xa];
                if constexpr (R > 0)
                    if (lane < 2 * R) q[i] = row[xb];
            }
            __syncthreads();  // the previous tile's readers are done
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                tile[(wave + i * kWaves) * kPitch + lane] = p[i];
                if constexpr (R > 0)
                    if (lane < 2 * R) tile[(wave + i * kWaves) * kPitch + 64 + lane] = q[i];
            }
        } else {
            // S(y, x) = input(x, y): a wave reads 64 pixels of one input row
            constexpr int kCols = (kSpan + kWaves - 1) / kWaves;
            const int y = min(y0 + lane, a.ho - 1);
            PixT p[kCols];
#pragma unroll
            for (int i = 0; i < kCols; ++i) {
                const int x = min(max(x0 - R + wave + i * kWaves, 0), a.wo - 1);
                p[i] = (img + (size_t)x * a.ws)[y];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kCols; ++i)
                if (wave + i * kWaves < kSpan) tile[lane * kPitch + wave + i * kWaves] = p[i];
        }
        __syncthreads();
        constexpr int kPer = 4;                      // outputs of a thread in a row
        constexpr int kRowsPass = kThreads / (kTile / kPer);
        const int cx = (threadIdx.x & (kTile / kPer - 1)) * kPer;
        const int x = x0 + cx;
#pragma unroll
        for (int ry = 0; ry < kTile; ry += kRowsPass) {
            const int ly = ry + (int)threadIdx.x / (kTile / kPer);
            const int* row = tile + ly * kPitch + cx;
            int s[kPer + 2 * R];
#pragma unroll
            for (int i = 0; i < kPer + 2 * R; ++i) s[i] = row[i];
            PixT o[kPer];
#pragma unroll
            for (int h = 0; h < kPer; ++h) {
                int acc = R > 0 ? 1 << (2 * R > 0 ? 2 * R - 1 : 0) : 0;  // half of 4^R
#pragma unroll
                for (int i = 0; i <= 2 * R; ++i) acc += binomial(2 * R, i) * s[h + i];
                o[h] = (PixT)(acc >> (2 * R));
            }
            if (y0 + ly >= a.ho || x >= a.wo) continue;
            PixT* dst = out + (size_t)(y0 + ly) * a.wo + x;
            if (a.vec && x + kPer <= a.wo) {
                if constexpr (sizeof(PixT) == 1) {
                    *reinterpret_cast<uint32_t*>(dst) = (uint32_t)o[0] | (uint32_t)o[1] << 8 |
                                                        (uint32_t)o[2] << 16 | (uint32_t)o[3] << 24;
                } else {
                    uint2 t;
                    t.x = (uint32_t)o[0] | (uint32_t)o[1] << 16;
                    t.y = (uint32_t)o[2] | (uint32_t)o[3] << 16;
                    *reinterpret_cast<uint2*>(dst) = t;
                }
            } else {
#pragma unroll
                for (int h = 0; h < kPer; ++h)
                    if (x + h < a.wo) dst[h] = o[h];
            }
        }
    }
}

template <typename PixT, int R>
void launch_prep_r(const PrepArgs& a, int transpose, dim3 grid, hipStream_t s) {
    if (transpose)
        hipLaunchKernelGGL((prep_kernel<PixT, R, true>), grid, dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((prep_kernel<PixT, R, false>), grid, dim3(kThreads), 0, s, a);
}

template <typename PixT>
void launch_prep_t(const PrepArgs& a, int radius, int transpose, dim3 grid, hipStream_t s) {
    switch (radius) {
        case 0: launch_prep_r<PixT, 0>(a, transpose, grid, s); return;
        case 1: launch_prep_r<PixT, 1>(a, transpose, grid, s); return;
        case 2: launch_prep_r<PixT, 2>(a, transpose, grid, s); return;
        case 3: launch_prep_r<PixT, 3>(a, transpose, grid, s); return;
        case 4: launch_prep_r<PixT, 4>(a, transpose, grid, s); return;
        case 5: launch_prep_r<PixT, 5>(a, transpose, grid, s); return;
        case 6: launch_prep_r<PixT, 6>(a, transpose, grid, s); return;
        default: launch_prep_r<PixT, 7>(a, transpose, grid, s); return;
    }
}

}  // namespace

hipError_t launch_prep(const void* img, int dtype, int h, int w, int radius, int transpose,
                       void* out, hipStream_t stream) {
    if (radius < 0 || radius > kMaxRadius) return hipErrorInvalidValue;
    PrepArgs a{};
    a.img = img;
    a.out = out;
    a.ws = w;
    a.ho = transpose ? w : h;
    a.wo = transpose ? h : w;
    const size_t four = dtype == 0 ? 4 : 8;  // bytes of four outputs
    a.vec = a.wo % 4 == 0 && reinterpret_cast<uintptr_t>(out) % four == 0;
    const int tiles_y = (a.ho + kTile - 1) / kTile;
    const dim3 grid((a.wo + kTile - 1) / kTile, tiles_y < 65535 ? tiles_y : 65535);
    TimedLaunch tl("prep_kernel", stream);
    if (dtype == 0)
        launch_prep_t<uint8_t>(a, radius, transpose, grid, stream);
    else
        launch_prep_t<uint16_t>(a, radius, transpose, grid, stream);
    return hipGetLastError();
}

}  // namespace fhtp
