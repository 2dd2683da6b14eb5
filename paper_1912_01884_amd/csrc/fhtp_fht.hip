// Band Fast Hough Transform for mostly vertical lines (Section 2.1).
//
// Every band of n = 2^p rows is zero-extended to the right by n columns and
// transformed with the dyadic shift-and-add recursion: stage j merges pairs of
// row blocks of 2^(j-1) rows into blocks of 2^j rows,
//
//   T_j(b, c, s) = T_{j-1}(2b, c, s/2) + T_{j-1}(2b+1, c + ceil(s/2), s/2)   (s/2 rounded down),
//
// so after p stages T_p(0, c, s) is the sum along the dyadic line that starts
// at column c and is displaced by s over the band.  Left-leaning lines are the
// same recursion on the band mirrored about its (cyclic) width, so both
// directions share one code path ("c-space": c = x for right-leaning lines,
// c = W-1-x for left-leaning ones).  Work per band and direction is p*n*W
// additions, the O((w + h/k) * (h/k) * log(h/k)) cost of Section 2.1.
//
// Layout on gfx950:
//   - short bands (at most 16 rows of 8-bit pixels, 32 of 16-bit ones),
//     fht_reg_kernel: one thread owns one c-space column and keeps the n
//     running sums of that column in VGPRs through all p stages; the operand
//     that comes from another column (c + ceil(s/2)) is exchanged through LDS
//     once per stage;
//   - taller ones, up to 256 rows, fht_split_kernel: the fine and the coarse levels of a group of shifts
//     run on lanes, and a sum goes through LDS once, in between;
//   - the rest: fht_split_kernel on 128-row sub-blocks, then
//     fht_combine_kernel adds the sub-blocks along the coarse levels.
// Global loads and table stores are coalesced along x.
#include <algorithm>
#include <atomic>
#include <type_traits>
#include <vector>

#include "fhtp_internal.h"

namespace fhtp {
namespace {

// Column offset of row y on the dyadic line of shift s over 2^p rows: bit
// (p-1-j) of y contributes ceil((s >> j) / 2).
__device__ __forceinline__ int dyadic_offset(int p, int s, int y) {
    int off = 0;
    for (int j = 0; j < p; ++j)
        if ((y >> (p - 1 - j)) & 1) off += (s >> (j + 1)) + ((s >> j) & 1);
    return off;
}

// Buffer resource over [base, base + bytes): loads beyond the extent read 0
// and stores beyond it are dropped by the hardware.  The third descriptor
// word selects 32-bit raw (untyped) access on the gfx9 family.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                             0x00020000);
}

template <typename PixT>
__device__ __forceinline__ uint32_t buffer_pixel(__amdgpu_buffer_rsrc_t r, unsigned int voff,
                                                 unsigned int soff) {
    if constexpr (sizeof(PixT) == 1)
        return __builtin_amdgcn_raw_buffer_load_b8(r, (int)voff, (int)soff, 0);
    else
        return __builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0);
}

// Stages 1 .. kLaneStages take their operands from lanes + 1 .. + 2^(J-1) of
// the wave instead of LDS (stage J reads columns c .. c + 2^(J-1)).
constexpr int kLaneStages = 2;

template <int P>
struct RegCfg {
    static constexpr int N = 1 << P;
    static constexpr int NT = 256;
    static constexpr int HALF = (N >= 2) ? N / 2 : 1;
    // Distinct columns of a workgroup: consecutive waves overlap by K columns
    // (see from_next_lane), so 64 - K per wave plus the last wave's K.
    static constexpr int K = (P >= 1) ? (1 << kLaneStages) - 1 : 0;
    static constexpr int NC = NT - (NT / 64 - 1) * K;
    // LDS holds the exchanged operands column by column: (column c, row r) at
    // c * RW + r.  RW is odd so that the 64 lanes of a wave, one column each,
    // hit distinct banks.  Reads reach column NC + HALF - 2; column NT + HALF
    // is the spare written by duplicate lanes.
    static constexpr int RW = (HALF >= 2) ? HALF + 1 : 1;
    static constexpr int SPARE = NT + HALF;
    static constexpr int LDS_WORDS = (N >= 2) ? (SPARE + 1) * RW : 1;
    static constexpr int NPK = (N + 1) / 2;            // packed 16-bit pixel pairs per column
    static constexpr int NDIR = (P == 0) ? 1 : 2;      // one-row bands have only d = 0
};

// The lower operands of shifts 2t and 2t+1 of one stage are the same lower-
// block sum T(2b+1, ., t) at columns c + t and c + t + 1 (ceil(s/2) in the
// recursion above).  A lane reads only the first from LDS and takes the second
// from lane + 1 of its wave with a DPP wave shift (lane 63 receives 0), which
// halves the LDS reads of a stage; the first kLaneStages stages need no LDS
// at all.  So that the lanes a column reads are in its own wave, consecutive
// waves overlap by K = 2^kLaneStages - 1 columns: lanes 64 - K .. 63 of wave q
// hold the columns of lanes 0 .. K - 1 of wave q + 1, only the latter copies
// are kept (the duplicates write their operands to a spare LDS column that no
// lane reads, and store nothing), and the last wave's top K lanes are halo.
__device__ __forceinline__ int32_t from_next_lane(int32_t x) {
    return __builtin_amdgcn_mov_dpp(x, 0x130 /* wave_shl:1 */, 0xf, 0xf, true);
}

// One stage of the recursion on the column held in v, in place: the operands
// of the lower half-blocks go through LDS, and outputs (2t, 2t+1) overwrite
// slots that no later t of the same stage still reads (t runs downwards).
// `col` is the thread's LDS column for reads, `wcol` the one it writes.
template <int N, int J, int RW>
__device__ __forceinline__ void fht_stage(int32_t (&v)[N], int32_t* lds, int col, int wcol) {
    constexpr int half = 1 << (J - 1);
    constexpr int blocks = N >> J;
    // The lane's LDS byte address, made opaque to the optimiser so that per-row
    // addresses are formed next to their use instead of being hoisted out of
    // the loop into one register per row.
    unsigned int lane_addr = (unsigned int)(col * RW) * 4u;
    __syncthreads();  // the previous stage's LDS reads are complete
#pragma unroll
    for (int b = 0; b < blocks; ++b)
#pragma unroll
        for (int t = 0; t < half; ++t) lds[wcol * RW + b * half + t] = v[b * 2 * half + half + t];
    __syncthreads();
    // Groups of at most 16 operand pairs, with scheduling barriers between
    // them, so the compiler cannot hoist every LDS read of the stage at once
    // (that would need 2n live registers).
    constexpr int G = half < 16 ? half : 16;
#pragma unroll
    for (int b = 0; b < blocks; ++b) {
#pragma unroll
        for (int g = half / G - 1; g >= 0; --g) {
            asm volatile("" : "+v"(lane_addr));
            const char* lbase = reinterpret_cast<const char*>(lds) + lane_addr;
#pragma unroll
            for (int t = g * G + G - 1; t >= g * G; --t) {
                const int32_t a = v[b * 2 * half + t];
                const int32_t x =
                    *reinterpret_cast<const int32_t*>(lbase + (t * RW + b * half + t) * 4);
                v[b * 2 * half + 2 * t + 1] = a + from_next_lane(x);
                v[b * 2 * half + 2 * t] = a + x;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

template <int N, int J, int P, int RW>
__device__ __forceinline__ void fht_stages(int32_t (&v)[N], int32_t* lds, int col, int wcol) {
    if constexpr (J <= P && J <= kLaneStages) {
        // Shifts 2t and 2t+1 add the lower block's shift t at columns c + t and
        // c + t + 1, i.e. lanes + t and + t + 1: moved by wave shifts, with no
        // LDS exchange and no barrier (the next LDS stage opens with one).
        constexpr int half = 1 << (J - 1);
#pragma unroll
        for (int b = 0; b < (N >> J); ++b) {
            int32_t o[2 * half];
#pragma unroll
            for (int t = 0; t < half; ++t) {
                const int32_t a = v[b * 2 * half + t];
                int32_t x = v[b * 2 * half + half + t];
#pragma unroll
                for (int q = 0; q < t; ++q) x = from_next_lane(x);
                o[2 * t] = a + x;
                o[2 * t + 1] = a + from_next_lane(x);
            }
#pragma unroll
            for (int q = 0; q < 2 * half; ++q) v[b * 2 * half + q] = o[q];
        }
        // The stage's sums are final here.  Integer adds reassociate freely, and
        // without this the compiler carries partial sums of several stages.
#pragma unroll
        for (int q = 0; q < N; ++q) asm volatile("" : "+v"(v[q]));
        fht_stages<N, J + 1, P, RW>(v, lds, col, wcol);
    } else if constexpr (J <= P) {
        fht_stage<N, J, RW>(v, lds, col, wcol);
        fht_stages<N, J + 1, P, RW>(v, lds, col, wcol);
    }
}

// One run of the register kernel for one image: its row blocks of 2^P rows,
// both directions, split into column tiles.  A launch takes a pack of runs
// (several images of the same band height) and numbers their work items
// consecutively from item0.
struct FhtJob {
    const void* img;  // first row of row block 0
    int32_t* out;     // tables [blocks][2n-1][W], or sub-block scratch
    uint16_t* out16;  // narrow tables: bands 0 .. narrow-1 as [narrow][2n-1][W] uint16
    int w, W;         // image width, table width (w + band height)
    int T, tiles;     // columns produced per tile, tiles per row block
    int item0;        // first work item of this run in the launch
    int to_table;     // 1: band tables; 0: c-space sub-block scratch
    int narrow;       // bands stored as uint16 (the rest, from band `narrow` on, go to out)
};

constexpr int kPack = 256;  // runs per launch (kernel arguments of up to 32 KB)
constexpr int kXcds = 8;   // accelerator dies of the MI355X, each with its own L2

// CAP runs per launch: 1 for a single image (small kernel arguments), kPack for batches.
template <int CAP>
struct FhtPack {
    FhtJob job[CAP];
    int count;  // runs in this pack
    int total;  // work items of the pack
    int first;  // split kernel: the item of this dispatch's first workgroup
};

// The run a work item belongs to (uniform across the workgroup).
template <int CAP>
__device__ __forceinline__ int fht_find_job(const FhtPack<CAP>& pk, int item) {
    // the last job whose first item is <= item (item0 ascends): binary search
    int lo = 0;
    if constexpr (CAP > 1) {
        int hi = pk.count - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pk.job[mid].item0 <= item)
                lo = mid;
            else
                hi = mid - 1;
        }
    }
    return lo;
}

struct FhtItem {
    int blk, dir, c, ximg;
    bool inside;
};

// Items of a row block alternate between the two directions, right-leaning
// tiles left to right and left-leaning tiles (whose c-space runs right to
// left in the image) in reverse, so consecutive items read overlapping image
// columns: right tile t and left tile tiles-1-t share most of their pixels.
template <int NDIR>
__device__ __forceinline__ FhtItem fht_decode(const FhtJob& J, int local, int col) {
    FhtItem it;
    const int per_blk = NDIR * J.tiles;
    it.blk = local / per_blk;
    const int u = local - it.blk * per_blk;
    it.dir = NDIR == 2 ? (u & 1) : 0;
    const int t = NDIR == 2 ? (u >> 1) : u;
    const int tile = it.dir ? J.tiles - 1 - t : t;
    it.c = tile * J.T + col;
    const int cm = it.c % J.W;
    it.ximg = it.dir == 0 ? cm : (J.W - 1 - cm);
    it.inside = it.ximg < J.w;
    return it;
}

// Pixels of one c-space column, two rows per 32-bit register.  The row block
// base is uniform (scalar registers), rows are scalar offsets, and the column
// is one 32-bit lane offset shared by every row.
template <int N, int NPK, int NDIR, typename PixT>
__device__ __forceinline__ void fetch_column(const FhtJob& J, int local, int col,
                                             uint32_t (&pk)[NPK]) {
    const FhtItem it = fht_decode<NDIR>(J, local, col);
    const PixT* img = static_cast<const PixT*>(J.img);
    const unsigned int row_bytes = (unsigned int)J.w * sizeof(PixT);
    const __amdgpu_buffer_rsrc_t r =
        make_rsrc(img + (size_t)it.blk * N * (size_t)J.w, (unsigned int)N * row_bytes);
    const unsigned int voff = (it.inside ? (unsigned int)it.ximg : 0u) * sizeof(PixT);
    // Row offsets advance in one scalar register that the optimiser cannot
    // precompute: it had hoisted every row's offset (of loads and of stores)
    // out of the item loop into scalar registers, and spilled them.
    unsigned int so = 0;
#pragma unroll
    for (int q = 0; q < NPK; ++q) {
        const uint32_t lo = buffer_pixel<PixT>(r, voff, so);
        uint32_t hi = 0u;
        if constexpr (N > 1) hi = buffer_pixel<PixT>(r, voff, so + row_bytes);
        pk[q] = it.inside ? (lo | (hi << 16)) : 0u;
        so += 2 * row_bytes;
        asm volatile("" : "+s"(so));
    }
}

// tables[blk][n-1 +- s][x] of a band of n = 2^P rows (d = 0 only from dir 0).
template <int P>
__device__ __forceinline__ void fht_store(const FhtJob& J, int local, int col,
                                          const int32_t (&v)[1 << P]) {
    using C = RegCfg<P>;
    constexpr int N = C::N;
    const FhtItem it = fht_decode<C::NDIR>(J, local, col);
    const int W = J.W;
    if (col >= J.T || it.c >= W) return;
    const unsigned int row_bytes = (unsigned int)W * 4u;
    if (it.blk < J.narrow) {
        // 16-bit table of a band whose line sums stay below 2^16
        constexpr int D = 2 * N - 1;
        const unsigned int row16 = (unsigned int)W * 2u;
        const unsigned int voff = (unsigned int)(it.dir == 0 ? it.c : (W - 1 - it.c)) * 2u;
        const __amdgpu_buffer_rsrc_t r =
            make_rsrc(J.out16 + (size_t)it.blk * D * (size_t)W, (unsigned int)D * row16);
        if (it.dir == 0) {
            unsigned int so = (unsigned int)(N - 1) * row16;
#pragma unroll
            for (int s = 0; s < N; ++s) {
                __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v[s], r, (int)voff, (int)so, 0);
                so += row16;
                asm volatile("" : "+s"(so));
            }
        } else {
            unsigned int so = (unsigned int)(N - 2) * row16;
#pragma unroll
            for (int s = 1; s < N; ++s) {
                __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v[s], r, (int)voff, (int)so, 0);
                so -= row16;
                asm volatile("" : "+s"(so));
            }
        }
    } else {
        constexpr int D = 2 * N - 1;
        const unsigned int voff = (unsigned int)(it.dir == 0 ? it.c : (W - 1 - it.c)) * 4u;
        const __amdgpu_buffer_rsrc_t r = make_rsrc(
            J.out + (size_t)(it.blk - J.narrow) * D * (size_t)W, (unsigned int)D * row_bytes);
        if (it.dir == 0) {
            unsigned int so = (unsigned int)(N - 1) * row_bytes;
#pragma unroll
            for (int s = 0; s < N; ++s) {
                __builtin_amdgcn_raw_buffer_store_b32(v[s], r, (int)voff, (int)so, 0);
                so += row_bytes;
                asm volatile("" : "+s"(so));
            }
        } else {
            unsigned int so = (unsigned int)(N - 2) * row_bytes;
#pragma unroll
            for (int s = 1; s < N; ++s) {
                __builtin_amdgcn_raw_buffer_store_b32(v[s], r, (int)voff, (int)so, 0);
                so -= row_bytes;
                asm volatile("" : "+s"(so));
            }
        }
    }
}

// Work item = (run, row block, direction, column tile).  The grid holds as
// many workgroups as the chip keeps resident and loops over the items, so a
// workgroup's table stores drain while it loads and transforms its next item,
// and it fetches the next item's pixels while the current one runs its stages.  A tile produces T columns (T <= NC - (n-1));
// the rest of its NC columns are halo.
template <int P, typename PixT, int CAP>
__global__ __launch_bounds__(RegCfg<P>::NT) void fht_reg_kernel(FhtPack<CAP> pk) {
    using C = RegCfg<P>;
    constexpr int N = C::N;
    __shared__ int32_t lds[C::LDS_WORDS];
    const int tid = threadIdx.x;
    const int total = pk.total;
    // The thread's column within the tile (waves overlap by K columns).
    const int col = (tid >> 6) * (64 - C::K) + (tid & 63);
    const bool wr = (tid & 63) < 64 - C::K || (tid >> 6) == C::NT / 64 - 1;  // not a duplicate
    const int wcol = wr ? col : C::SPARE;

    uint32_t pre[C::NPK];
    // Workgroups are spread over the XCDs round-robin (workgroup b on XCD
    // b % 8).  Each XCD is given a contiguous run of items instead, so the
    // tiles that share pixel columns meet in one L2: slot i of the launch
    // (workgroup i % grid, round i / grid) takes item xmap(i), which lies in
    // the run of XCD i % 8 whenever the grid is a multiple of 8 or covers
    // every item in one round.
    auto xmap = [total](int i) {
        const int xcd = i % kXcds, slot = i / kXcds;
        return xcd * (total / kXcds) + min(xcd, total % kXcds) + slot;
    };
    const int grid = (int)gridDim.x;
    int vi = blockIdx.x;
    int item = xmap(vi);
    {
        const int j = fht_find_job(pk, item);
        fetch_column<N, C::NPK, C::NDIR, PixT>(pk.job[j], item - pk.job[j].item0, col, pre);
    }
    while (vi < total) {
        const int j = fht_find_job(pk, item);
        const FhtJob& J = pk.job[j];
        const int local = item - J.item0;
        int32_t v[N];
#pragma unroll
        for (int q = 0; q < C::NPK; ++q) {
            v[2 * q] = (int32_t)(pre[q] & 0xffffu);
            if (2 * q + 1 < N) v[2 * q + 1] = (int32_t)(pre[q] >> 16);
        }
        vi += grid;
        {
            // Unconditional prefetch (the last round re-reads its own item).
            const int nx = vi < total ? xmap(vi) : item;
            const int jn = fht_find_job(pk, nx);
            fetch_column<N, C::NPK, C::NDIR, PixT>(pk.job[jn], nx - pk.job[jn].item0, col, pre);
        }

        if constexpr (sizeof(PixT) == 1 && P >= 2) {
            // Stages 1 .. p-1 never mix the top and bottom halves of the
            // block, and apply the same shifts to both.  With 8-bit pixels a
            // half's sums stay below 2^16 (at most 8 * 255), so row y and row
            // y + n/2 share a register (low and high 16 bits, no carry between
            // them) and those stages run as the recursion of a block of n/2
            // rows on n/2 registers: half the LDS exchange and half the adds.
            constexpr int H = N / 2;
            int32_t pk[H];
#pragma unroll
            for (int y = 0; y < H; ++y) pk[y] = v[y] | (v[y + H] << 16);
            fht_stages<H, 1, P - 1, C::RW>(pk, lds, col, wcol);
#pragma unroll
            for (int t = 0; t < H; ++t) {
                v[t] = pk[t] & 0xffff;
                v[t + H] = (int32_t)((uint32_t)pk[t] >> 16);
            }
            fht_stages<N, P, P, C::RW>(v, lds, col, wcol);  // the last stage, unpacked
        } else {
            fht_stages<N, 1, P, C::RW>(v, lds, col, wcol);
        }
        if (wr) fht_store<P>(J, local, col, v);
        if (vi < total) item = xmap(vi);
    }
}

// ---- bands of 2^5 .. 2^8 rows ---------------------------------------------------
//
// The shifts s of a band are taken in groups that share their top Q bits g.
// Inside a group the recursion splits into three parts:
//
//   - the first Q levels see only s >> (p-Q) .. = g, one line per block: R =
//     2^Q rows are summed along the dyadic line of shift g (base sums);
//   - the fine levels make, from NF = 2^LF base sums, the NF lines whose next
//     LF bits are f.  Writing the shift at fine level j as g 2^j + f_j, its
//     operand offset is g 2^(j-1) + ceil(f_j / 2): the first part adds up, over
//     the levels, to g per base sum, so with base sum q read g q columns to the
//     right what remains is the recursion of an NF-row band (shifts f_j);
//   - the coarse levels join the M = 8 blocks of NF base sums in the same way:
//     with block m of fine shift f read (g NF + f) m columns to the right, what
//     remains is the recursion of an 8-row band, whose 8 shifts e are the
//     band's shifts s = (g NF + f) 8 + e.
//
// So a workgroup makes one group of shifts of a column tile: phase 1 loads the
// pixels at their skewed columns (a lane a column) and leaves the fine sums in
// LDS; phase 2 reads them once at theirs (a lane two columns) and stores the 8
// finished rows of a (g, f).  The small recursions run on lanes (a shift by a
// column is a DPP wave shift), so a sum goes through LDS once, against once per
// level in fht_reg_kernel, with one barrier, and no lane holds more than a few
// dozen registers: two workgroups of 16 waves share a CU, and one's loads and
// sums run beside the other's stores.  Its cost is that every group of shifts
// reads the pixels again (from L1 and L2), that a wave's 64 columns give 57 (the
// residual shifts reach 7 columns) and that a tile of 228 needs the fine sums
// of 285.
//
// What bounds it: at 4096 x 4096, n = 128, 16-bit pixels (171 MB in and out)
// 50 us a launch, 3.4 TB/s (fht_reg_kernel, one workgroup of 8 waves a CU on 147
// KB of LDS: 63.5 us).  Timing copies: without the stores 31 us, without the
// loads 37, phase 2 and its stores alone 28, phase 2 alone 15; so the stores
// drain beside about half of the rest.  Streaming stores run in 42 us, but the
// tables then miss the memory-side cache when the DP reads them (a detection
// 177 against 171 us).  Two columns a lane in phase 1 (pairs of pixels from
// aligned addresses, put in place with the next lane's) took 65 us, eight waves
// a workgroup 58.
//
// 8-bit pixels (BOTH): a lane's register holds the right-leaning line's sum in its
// low half and the left-leaning line's in its high half (both directions are
// the same recursion in c-space, at the same c) up to the last level (sums of at
// most 64 rows, 64 * 255 < 2^16: no carry between the halves), which runs on 32
// bits apart.  Bands of at most 128 rows.
template <int P>
struct SplitCfg {
    static constexpr int N = 1 << P;
    static constexpr int LF = P >= 6 ? 3 : P - 3;  // fine levels
    static constexpr int NF = 1 << LF;             // fine shifts (and base sums) of a block
    static constexpr int Q = P - 3 - LF;           // levels in a base sum
    static constexpr int R = 1 << Q;               // rows in a base sum
    static constexpr int G = 1 << Q;               // groups of shifts
    static constexpr int M = 8;                    // blocks
    // 512 threads for 256-row bands, for the int32 tables of large 8-bit images: us of the
    // band tables of 8192 x 16384 476, with 1024 threads 532 (4096 x 16384 242 / 267).
    // Elsewhere 1024 would be the faster: in detections of 4096 x 4096 61.3 / 56.4 of 8-bit
    // and 74.9 / 71.0 of 16-bit pixels, of 8192 x 16384 406 / 395 and 531 / 535.
    static constexpr int NT = P <= 7 ? 1024 : 512;
    static constexpr int ROWS = NF * R;            // rows of a block
    static constexpr int WC = 57;                  // columns a wave of phase 1 makes
    static constexpr int CG = 5;                   // waves of phase 1 across
    // columns a workgroup produces, in two waves' halves: what CG WC leaves
    // after the skew f m and the residual shifts
    static constexpr int FIT = (CG * WC - (NF - 1) * (M - 1) - 7) / 4 * 4;
    static constexpr int TC = FIT < 240 ? FIT : 240;  // (120 of a half wave's 128 are whole)
    static constexpr int HC = TC / 2;
    static constexpr int PITCH = CG * WC + 8;      // (a half wave reads past its columns)
};

// One level of the recursion on the COLS (1 or 2) adjacent columns of a lane,
// in place, shifts in order: the lower half-block's shift t is read t and t + 1
// columns to the right.
template <int ROWS, int COLS, int J>
__device__ __forceinline__ void lane_stage(int32_t (&v)[ROWS][COLS]) {
    constexpr int half = 1 << (J - 1);
    // the columns one to the right
    auto next = [](int32_t(&y)[COLS]) {
        const int32_t z = from_next_lane(y[0]);
        if constexpr (COLS == 2) y[0] = y[1];
        y[COLS - 1] = z;
    };
#pragma unroll
    for (int b = 0; b < (ROWS >> J); ++b) {
        int32_t o[2 * half][COLS];
#pragma unroll
        for (int t = 0; t < half; ++t) {
            const int32_t(&a)[COLS] = v[b * 2 * half + t];
            int32_t y[COLS];
#pragma unroll
            for (int h = 0; h < COLS; ++h) y[h] = v[b * 2 * half + half + t][h];
#pragma unroll
            for (int q = 0; q < t; ++q) next(y);
#pragma unroll
            for (int h = 0; h < COLS; ++h) o[2 * t][h] = a[h] + y[h];
            next(y);
#pragma unroll
            for (int h = 0; h < COLS; ++h) o[2 * t + 1][h] = a[h] + y[h];
        }
#pragma unroll
        for (int q = 0; q < 2 * half; ++q)
#pragma unroll
            for (int h = 0; h < COLS; ++h) v[b * 2 * half + q][h] = o[q][h];
    }
    // final here, as in fht_stages
#pragma unroll
    for (int q = 0; q < ROWS; ++q)
#pragma unroll
        for (int h = 0; h < COLS; ++h) asm volatile("" : "+v"(v[q][h]));
}

template <int ROWS, int COLS, int FROM, int TO>
__device__ __forceinline__ void lane_stages(int32_t (&v)[ROWS][COLS]) {
    if constexpr (FROM <= TO) {
        lane_stage<ROWS, COLS, FROM>(v);
        lane_stages<ROWS, COLS, FROM + 1, TO>(v);
    }
}

// One item of the split kernel: a group of shifts g of a column tile (first
// column ct) of row block blk, in direction dir (8-bit pixels: both).
struct SplitItem {
    int job, blk, dir, g, ct;
};

// The pixels of one wave of phase 1: the rows of block m at c-space column cb +
// lane, base sum q read g (NF m + q) columns to its right (cb uniform); p[i]
// of row i; with BOTH the right-leaning column's in p[i] and the left-leaning
// one's in p[ROWS + i].
template <int P, bool BOTH, typename PixT>
__device__ __forceinline__ void split_load(const FhtJob& J, const SplitItem& it, int m, int cb,
                                           uint32_t (&p)[SplitCfg<P>::ROWS * (BOTH ? 2 : 1)]) {
    using C = SplitCfg<P>;
    constexpr int ROWS = C::ROWS;
    constexpr int sz = (int)sizeof(PixT);
    const int lane = threadIdx.x & 63;
    const int w = J.w, W = J.W, g = it.g, dir = it.dir;
    const int step = w * sz;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(
        static_cast<const char*>(J.img) + ((size_t)it.blk * C::N + (size_t)m * ROWS) * (size_t)step,
        (unsigned int)(ROWS * step));
    // skew of row i of the block (i = ROWS: of the next block's first row)
    auto skew = [&](int i) { return g * (i / C::R) + dyadic_offset(C::Q, g, i % C::R); };
    const int cm = cb + g * C::NF * m;
    const int reach = 63 + g * C::NF;          // to the last column any row reads
    const bool in_right = cm + reach < w;      // every column is a pixel of the image
    const bool in_left = cm >= W - w && cm + reach < W;
    if (BOTH ? in_right && in_left : dir ? in_left : in_right) {
        // one lane offset, rows and skews in the scalar offset
        const int vr = lane * sz, vl = (63 - lane) * sz;
        int ar = cm * sz, al = (W - 1 - 63 - cm) * sz;
        if constexpr (BOTH) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                p[i] = buffer_pixel<PixT>(rs, (unsigned)vr, (unsigned)ar);
                p[ROWS + i] = buffer_pixel<PixT>(rs, (unsigned)vl, (unsigned)al);
                const int d = (skew(i + 1) - skew(i)) * sz;
                ar += step + d;
                al += step - d;
                asm volatile("" : "+s"(ar), "+s"(al));
            }
        } else {
            const int vo = dir ? vl : vr, sg = dir ? -1 : 1;
            int at = dir ? al : ar;
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                p[i] = buffer_pixel<PixT>(rs, (unsigned)vo, (unsigned)at);
                at += step + sg * (skew(i + 1) - skew(i)) * sz;
                asm volatile("" : "+s"(at));
            }
        }
    } else {
        // Byte offset of the pixel of c-space column c < 2 W; past the view
        // outside the image, where loads return 0.
        auto at = [&](int c, bool left) -> unsigned int {
            const int cc = c >= W ? c - W : c;
            const int x = left ? W - 1 - cc : cc;
            return (unsigned)x < (unsigned)w ? (unsigned int)(x * sz) : 0x80000000u;
        };
        unsigned int so = 0;
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int c = cm + lane + skew(i);
            p[i] = buffer_pixel<PixT>(rs, at(c, !BOTH && dir), so);
            if constexpr (BOTH) p[ROWS + i] = buffer_pixel<PixT>(rs, at(c, true), so);
            so += (unsigned int)step;
            asm volatile("" : "+s"(so));
        }
    }
}

// The fine sums v[f] of those pixels.
template <int P, bool BOTH, typename PixT>
__device__ __forceinline__ void split_fine(const uint32_t (&p)[SplitCfg<P>::ROWS * (BOTH ? 2 : 1)],
                                           int32_t (&v)[SplitCfg<P>::NF][1]) {
    using C = SplitCfg<P>;
#pragma unroll
    for (int i = 0; i < C::ROWS; ++i) {
        uint32_t t = p[i];
        if constexpr (BOTH) t |= p[C::ROWS + i] << 16;
        v[i / C::R][0] = i % C::R == 0 ? (int32_t)t : v[i / C::R][0] + (int32_t)t;
    }
    lane_stages<C::NF, 1, 1, C::LF>(v);
}

// The finished rows s = s0 .. s0 + 7 of one direction at tile columns c, c + 1
// (those below `lim`), to the table or the sub-block scratch.
template <int P, bool E16, bool REV>
__device__ __forceinline__ void split_rows(char* base, int W, int x, bool two, bool skip0,
                                           const int32_t (&v)[8][2]) {
    constexpr int esz = E16 ? 2 : 4;
    const unsigned int row = (unsigned int)W * esz;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(base, 8u * row);
    unsigned int so = REV ? 7u * row : 0u;
    const int xa = (REV && two ? x - 1 : x) * esz;
    // Rows with the pair stores of even e and of odd e aligned or not (16-bit
    // elements: one aligned 32-bit store, or two of 16 bits).
    auto rows = [&](auto even_ok, auto odd_ok) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (e > 0 || !skip0) {
                const uint32_t a = (uint32_t)v[e][REV ? 1 : 0], b = (uint32_t)v[e][REV ? 0 : 1];
                const bool ok = (e & 1) ? decltype(odd_ok)::value : decltype(even_ok)::value;
                if (!two) {
                    const uint32_t o = (uint32_t)v[e][0];
                    if constexpr (E16)
                        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)o, rs, xa, (int)so, 0);
                    else
                        __builtin_amdgcn_raw_buffer_store_b32(o, rs, xa, (int)so, 0);
                } else if constexpr (!E16) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    u32x2 t;
                    t.x = a;
                    t.y = b;
                    __builtin_amdgcn_raw_buffer_store_b64(t, rs, xa, (int)so, 0);
                } else if (ok) {
                    __builtin_amdgcn_raw_buffer_store_b32(a | (b << 16), rs, xa, (int)so, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)a, rs, xa, (int)so, 0);
                    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)b, rs, xa + 2, (int)so, 0);
                }
            }
            so = REV ? so - row : so + row;
        }
    };
    if (E16 && two) {
        // the parity of a row's pairs is the same on every lane (c is even)
        const int first = __builtin_amdgcn_readfirstlane(
            (int)(((uint32_t)reinterpret_cast<uintptr_t>(base) + (uint32_t)xa) >> 1));
        const bool ok0 = ((first + (REV ? 7 : 0) * W) & 1) == 0;
        const bool ok1 = ((first + (REV ? 6 : 1) * W) & 1) == 0;
        if (ok0 && ok1)
            rows(std::true_type{}, std::true_type{});
        else if (ok0)
            rows(std::true_type{}, std::false_type{});
        else if (ok1)
            rows(std::false_type{}, std::true_type{});
        else
            rows(std::false_type{}, std::false_type{});
    } else {
        rows(std::true_type{}, std::true_type{});
    }
}

template <int P, bool E16, bool REV>
__device__ __forceinline__ void split_cols(char* base, int W, int ct, int c, int lim, bool skip0,
                                           const int32_t (&v)[8][2]) {
    const int x = REV ? W - 1 - (ct + c) : ct + c;
    if (c + 1 < lim)
        split_rows<P, E16, REV>(base, W, x, true, skip0, v);
    else if (c < lim)  // the last column of an odd tile
        split_rows<P, E16, REV>(base, W, x, false, skip0, v);
}

template <int P, typename PixT>
__device__ __forceinline__ void split_store(const FhtJob& J, int blk, int dir, int s0, int ct, int c,
                                            int lim, const int32_t (&v)[8][2]) {
    constexpr int N = 1 << P, D = 2 * N - 1;
    const int W = J.W;
    // The 8 rows' first one in memory: rows N-1 + s or, leaning left, N-1 - s
    // of the table; row s of the scratch.
    if (J.to_table) {
        const bool skip0 = dir && s0 == 0;  // displacement 0 comes from the right-leaning lines
        const int row = dir ? N - 1 - s0 - 7 : N - 1 + s0;
        if constexpr (sizeof(PixT) == 1) {
            if (blk < J.narrow) {
                char* base = reinterpret_cast<char*>(J.out16 + ((size_t)blk * D + row) * (size_t)W);
                if (dir)
                    split_cols<P, true, true>(base, W, ct, c, lim, skip0, v);
                else
                    split_cols<P, true, false>(base, W, ct, c, lim, false, v);
                return;
            }
        }
        char* base =
            reinterpret_cast<char*>(J.out + ((size_t)(blk - J.narrow) * D + row) * (size_t)W);
        if (dir)
            split_cols<P, false, true>(base, W, ct, c, lim, skip0, v);
        else
            split_cols<P, false, false>(base, W, ct, c, lim, false, v);
    } else if constexpr (P == kRegMaxP) {
        const size_t at = (((size_t)blk * 2 + dir) * N + s0) * (size_t)W;
        if constexpr (sizeof(PixT) == 1)
            split_cols<P, true, false>(reinterpret_cast<char*>(J.out) + at * 2, W, ct, c, lim, false, v);
        else
            split_cols<P, false, false>(reinterpret_cast<char*>(J.out) + at * 4, W, ct, c, lim, false, v);
    }
}

// Item of workgroup b of the pack.  Workgroup b runs on XCD b % 8; each XCD
// is dealt runs of kRun items, so that those that share pixel columns meet in
// one L2 while the chip as a whole writes along one band at a time.  (Each XCD
// on a contiguous eighth of the items, eight bands far apart being written at
// once: 54.9 against 49.9 us at 4096 x 4096, n = 128, 16-bit pixels, 829
// against 776 at 16384 x 16384; runs of 4: 50.4 and 813, of 64: 50.0 and 764.)
// Tiles go from both ends in turn, as a left-leaning tile t covers the image
// columns of right-leaning tile tiles - 1 - t.
constexpr int kRun = 16;

template <int P, bool BOTH, int CAP>
__device__ __forceinline__ SplitItem split_item(const FhtPack<CAP>& pk, int b) {
    using C = SplitCfg<P>;
    const int xcd = b % kXcds, slot = b / kXcds;
    const int whole = pk.total / (kXcds * kRun) * (kXcds * kRun);
    const int item = b < whole ? slot / kRun * (kXcds * kRun) + xcd * kRun + slot % kRun : b;
    SplitItem it;
    it.job = __builtin_amdgcn_readfirstlane(fht_find_job(pk, item));
    const FhtJob& J = pk.job[it.job];
    int local = item - J.item0;
    const int per_blk = (BOTH ? 1 : 2) * C::G * J.tiles;
    it.blk = local / per_blk;
    local -= it.blk * per_blk;
    it.g = local & (C::G - 1);
    const int u = local >> C::Q;
    it.dir = BOTH ? 0 : u & 1;
    const int tile = (u & 1) ? J.tiles - 1 - (u >> 1) : u >> 1;
    it.ct = tile * J.T;
    return it;
}

template <int P, bool BOTH, typename PixT, int CAP>
__global__ __launch_bounds__(SplitCfg<P>::NT, SplitCfg<P>::NT / 128) void fht_split_kernel(FhtPack<CAP> pk) {
    using C = SplitCfg<P>;
    constexpr int WAVES = C::NT / 64;
    __shared__ int32_t fine[C::M * C::NF * C::PITCH];  // [m][f][column]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const SplitItem it = split_item<P, BOTH>(pk, pk.first + (int)blockIdx.x);
    const FhtJob& J = pk.job[it.job];
    // Phase 1: a wave per (block, CG-th of the columns).  (The pixels of all
    // of a wave's tasks loaded before the first one's sums: 53.6 against 50.1 us
    // at 4096 x 4096, n = 128, 16-bit pixels.  The loads are not what it waits for.)
    // A wave stays with one block, so its rows' view and skews are formed once;
    // unrolled, 78.8 -> 74.6 us at 4096 x 4096, n = 256, 16-bit, 50.8 -> 49.0 at 128.
    static_assert(WAVES % C::M == 0, "whole rounds of the blocks");
    const int m = wave % C::M;
#pragma unroll
    for (int q = 0; q < (C::M * C::CG + WAVES - 1) / WAVES; ++q) {
        const int cg = wave / C::M + q * (WAVES / C::M);
        if (cg >= C::CG) break;
        uint32_t px[C::ROWS * (BOTH ? 2 : 1)];
        split_load<P, BOTH, PixT>(J, it, m, it.ct + cg * C::WC, px);
        int32_t v[C::NF][1];
        split_fine<P, BOTH, PixT>(px, v);
        if (lane < C::WC) {
#pragma unroll
            for (int f = 0; f < C::NF; ++f)
                fine[(m * C::NF + f) * C::PITCH + cg * C::WC + lane] = v[f][0];
        }
    }
    __syncthreads();
    // Phase 2: a wave per (f, half of the tile).
    const int lim = min(J.T, J.W - it.ct);
#pragma unroll 1
    for (int task = wave; task < C::NF * 2; task += WAVES) {
        const int f = task % C::NF, og = task / C::NF;
        const int c = og * C::HC + 2 * lane;
        int32_t v[8][2];
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int32_t* src = &fine[(m * C::NF + f) * C::PITCH + c + f * m];
            v[m][0] = src[0];
            v[m][1] = src[1];
        }
        const int s0 = (it.g * C::NF + f) * 8;
        const bool st = 2 * lane < C::HC;
        if constexpr (BOTH) {
            lane_stages<8, 2, 1, 2>(v);
            int32_t r[8][2];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                r[e][0] = v[e][0] & 0xffff;
                r[e][1] = v[e][1] & 0xffff;
                v[e][0] = (int32_t)((uint32_t)v[e][0] >> 16);
                v[e][1] = (int32_t)((uint32_t)v[e][1] >> 16);
            }
            lane_stages<8, 2, 3, 3>(r);
            if (st) split_store<P, PixT>(J, it.blk, 0, s0, it.ct, c, lim, r);
            lane_stages<8, 2, 3, 3>(v);
            if (st) split_store<P, PixT>(J, it.blk, 1, s0, it.ct, c, lim, v);
        } else {
            lane_stages<8, 2, 1, 3>(v);
            if (st) split_store<P, PixT>(J, it.blk, it.dir, s0, it.ct, c, lim, v);
        }
    }
}

// Pass 2 for bands of n = 2^p > 2^8 rows: the band is M = n/128 sub-blocks whose
// FHTs (fine shift sf = s >> (p-7)) sit in `sub`; the line of shift s starts in
// sub-block m at c + D_s(m*128), so T(c, s) = sum_m sub[m][sf][(c + D_s(128 m)) mod W].
// A workgroup covers 256 columns of one (band, direction) for kShiftGroup
// consecutive shifts; the offsets D_s(128 m) are uniform (scalar) per shift.
struct CombineJob {
    const void* sub;   // [sub-blocks][2][128][W] int32, or uint16 for 8-bit pixels (sub16)
    int32_t* tables;   // wide bands (from band `narrow` on), [.][2n-1][W] int32
    uint16_t* tab16;   // narrow bands 0 .. narrow-1, [.][2n-1][W] uint16
    int p, W, k, tiles_x;
    int item0;
    int narrow;
    int sub16;
};

struct CombinePack {
    CombineJob job[kPack];
    int count;
    int total;
};

constexpr int kShiftGroup = 16;

// dyadic_offset(7 + SH, s, m << 7): only the bits of m are set in the row, and
// bit b of m is row bit 7 + b, i.e. j = SH - 1 - b of the closed form.  Every
// shift is a constant, so the offsets cost a handful of scalar operations.
template <int SH>
__device__ __forceinline__ int sub_block_offset(int s, int m) {
    int off = 0;
#pragma unroll
    for (int b = 0; b < SH; ++b)
        if ((m >> b) & 1) off += (s >> (SH - b)) + ((s >> (SH - 1 - b)) & 1);
    return off;
}

// SH = p - 7, M = 2^SH sub-blocks per band; SubT: the scratch's cell type.
template <int SH, typename SubT>
__global__ __launch_bounds__(256) void fht_combine_kernel(CombinePack pk) {
    constexpr int M = 1 << SH;
    const int item = blockIdx.x;
    int j = 0;
    for (int hi = pk.count - 1; j < hi;) {  // last job with item0 <= item
        const int mid = (j + hi + 1) >> 1;
        if (pk.job[mid].item0 <= item)
            j = mid;
        else
            hi = mid - 1;
    }
    const CombineJob& J = pk.job[j];
    const int p = J.p;
    const int n = 1 << p;
    const int D = 2 * n - 1;
    const int W = J.W;
    const int groups = n / kShiftGroup;
    int local = item - J.item0;  // ((band * 2 + dir) * groups + g) * tiles_x + tile
    const int tile = local % J.tiles_x;
    local /= J.tiles_x;
    const int g = local % groups;
    const int bd = local / groups;
    const int dir = bd & 1;
    const int band = bd >> 1;
    const int c = tile * 256 + threadIdx.x;
    if (c >= W) return;
    const size_t row = (size_t)W;
    const SubT* base = static_cast<const SubT*>(J.sub) + (size_t)band * M * 2 * (1 << kRegMaxP) * row;
    const bool n16 = band < J.narrow;
    int32_t* out = J.tables + (size_t)(band - J.narrow) * D * row;
    uint16_t* out16 = J.tab16 + (size_t)band * D * row;
    const int xo = dir == 0 ? c : (W - 1 - c);
    // Every load of the workgroup's shifts first (all in flight together),
    // then the sums and the stores.
    int32_t acc[kShiftGroup];
#pragma unroll
    for (int t = 0; t < kShiftGroup; ++t) {
        const int s = g * kShiftGroup + t;
        const int sf = s >> SH;
        int32_t a = 0;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            int cc = c + sub_block_offset<SH>(s, m);
            cc -= cc >= W ? W : 0;  // offsets are below n < W, so one wrap at most
            a += (int32_t)base[((size_t)(m * 2 + dir) * (1 << kRegMaxP) + sf) * row + cc];
        }
        acc[t] = a;
    }
#pragma unroll
    for (int t = 0; t < kShiftGroup; ++t) {
        const int s = g * kShiftGroup + t;
        if (dir == 1 && s == 0) continue;
        const int r = dir == 0 ? (n - 1 + s) : (n - 1 - s);
        if (n16)
            out16[(size_t)r * row + xo] = (uint16_t)acc[t];
        else
            out[(size_t)r * row + xo] = acc[t];
    }
}

constexpr int kMaxDevices = 64;

int current_device() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return 0;
    }
    return dev;
}

// Compute units of the current device, queried once per device.
int device_cus() {
    static std::atomic<int> cus[kMaxDevices];
    const int dev = current_device();
    int c = cus[dev].load(std::memory_order_relaxed);
    if (c <= 0) {
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            c <= 0) {
            (void)hipGetLastError();
            c = 256;
        }
        cus[dev].store(c, std::memory_order_relaxed);
    }
    return c;
}

// One register-kernel run to schedule (host side).
struct RegRun {
    const void* img;
    int dtype, p;   // pixel type, log2 of the row-block height the kernel runs
    int w, W, blocks, to_table;
    int32_t* out;
    uint16_t* out16;
    int narrow;
    int grid_mode;  // 0: resident grid; 1: one workgroup per item
};

template <int P, typename PixT, int CAP>
hipError_t launch_reg_pack(const RegRun* runs, int count, hipStream_t stream) {
    using C = RegCfg<P>;
    // resident workgroups per CU for this instantiation, per device
    static std::atomic<int> occ_of[kMaxDevices];
    const int dev = current_device();
    int occupancy = occ_of[dev].load(std::memory_order_relaxed);
    if (occupancy <= 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occupancy, fht_reg_kernel<P, PixT, CAP>,
                                                         C::NT, 0) != hipSuccess ||
            occupancy <= 0) {
            (void)hipGetLastError();
            occupancy = 1;
        }
        occ_of[dev].store(occupancy, std::memory_order_relaxed);
    }
    const int Tmax = C::NC - (C::N - 1);
    FhtPack<CAP> pk{};
    long long total = 0;
    for (int q = 0; q < count; ++q) {
        const RegRun& r = runs[q];
        // Tile width: the fewest tiles per row block of at most Tmax columns,
        // spread evenly so every tile does about the same work.
        const int tiles = (r.W + Tmax - 1) / Tmax;
        FhtJob& J = pk.job[q];
        J.img = r.img;
        J.out = r.out;
        J.w = r.w;
        J.W = r.W;
        J.tiles = tiles;
        J.T = (r.W + tiles - 1) / tiles;
        J.item0 = (int)total;
        J.to_table = r.to_table;
        J.out16 = r.out16;
        J.narrow = r.narrow;
        total += (long long)tiles * r.blocks * C::NDIR;
        if (total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    }
    pk.count = count;
    pk.total = (int)total;
    if (total == 0) return hipSuccess;
    // Resident grid (as many workgroups as the chip keeps, looping over the
    // items) unless the pack asks for one workgroup per item.
    const long long slots = runs[0].grid_mode ? total : (long long)occupancy * device_cus();
    const int grid = (int)(total < slots ? total : slots);
    {
        TimedLaunch tl("fht_reg_kernel", stream);
        hipLaunchKernelGGL((fht_reg_kernel<P, PixT, CAP>), dim3(grid), dim3(C::NT), 0, stream, pk);
    }
    return hipGetLastError();
}

template <int P, bool BOTH, typename PixT, int CAP>
hipError_t launch_split_as(const RegRun* runs, int count, hipStream_t stream) {
    using C = SplitCfg<P>;
    FhtPack<CAP> pk{};
    long long total = 0;
    for (int q = 0; q < count; ++q) {
        const RegRun& r = runs[q];
        // The fewest tiles of at most TC columns, of equal (even) width.
        const int tiles = (r.W + C::TC - 1) / C::TC;
        FhtJob& J = pk.job[q];
        J.img = r.img;
        J.out = r.out;
        J.w = r.w;
        J.W = r.W;
        J.tiles = tiles;
        J.T = ((r.W + tiles - 1) / tiles + 1) & ~1;
        J.item0 = (int)total;
        J.to_table = r.to_table;
        J.out16 = r.out16;
        J.narrow = r.narrow;
        total += (long long)tiles * r.blocks * C::G * (BOTH ? 1 : 2);
        if (total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    }
    pk.count = count;
    pk.total = (int)total;
    if (total == 0) return hipSuccess;
    // One workgroup per item: its stores drain while others load (a resident
    // grid looping over the items makes an item's loads wait for the stores of
    // the one before: 57.5 against 53.9 us at 4096 x 4096, n = 128, 16 bits).
    hipError_t e = hipSuccess;
    for_each_dispatch(total, C::NT, [&](int first, int groups) {
        if (e != hipSuccess) return;
        pk.first = first;
        TimedLaunch tl("fht_reg_kernel", stream);  // one family: the band transform
        hipLaunchKernelGGL((fht_split_kernel<P, BOTH, PixT, CAP>), dim3((unsigned)groups), dim3(C::NT), 0,
                           stream, pk);
        e = hipGetLastError();
    });
    return e;
}

// 8-bit pixels: both directions in a workgroup, but one for 256-row bands (4096 x
// 4096 85.3 / 68.8 us) and where both would leave the chip's workgroup slots (two
// a CU) idle.  Both / one, us in a detection: 80
// items (1024 x 1024, n = 64) 10.1 / 8.5, 96 (n = 128) 11.9 / 9.3, 320 (2048 x
// 2048, n = 128) 18.3 / 16.2, 352 (2048 x 2047, n = 256) 35.1 / 32.5, but 448
// (2048 x 3000, n = 64) 14.1 / 15.3 and 1184 (4096 x 4096, n = 128) 37.4 / 40.3.
constexpr long long kOneWayItems = 384;

template <int P, typename PixT, int CAP>
hipError_t launch_split_pack(const RegRun* runs, int count, hipStream_t stream) {
    using C = SplitCfg<P>;
    if constexpr (sizeof(PixT) == 1 && P <= 7) {
        long long items = 0;
        for (int q = 0; q < count; ++q)
            items += (long long)((runs[q].W + C::TC - 1) / C::TC) * runs[q].blocks * C::G;
        if (items > kOneWayItems) return launch_split_as<P, true, PixT, CAP>(runs, count, stream);
    }
    return launch_split_as<P, false, PixT, CAP>(runs, count, stream);
}

// Largest band height (as a power of two) made in one pass, and the smallest
// one the split kernel takes.  Measured at 4096 x 4096 (us; split, then the
// register kernel or the two passes):
//   8-bit:  n = 32 32.5 / 35.4, 64 30.3 / 38.6, 128 42.1 / 43.7 (15.1 / 17.2 at
//           1024 x 1024), 256 (a direction a workgroup) 68.8 / 74.5;
//   16-bit: n = 32 54.1 / 43.4, but 64 45.1 / 56.7, 128 50.3 / 59.0, 256 81 /
//           95, 512 128 / 105 alone: every group of shifts loads the pixels again.
constexpr int kOnePassMax = 8;
constexpr int split_min(int dtype) { return dtype == 0 ? 5 : 6; }

template <int P, typename PixT, int CAP>
hipError_t launch_one(const RegRun* runs, int count, hipStream_t stream) {
    constexpr int dtype = sizeof(PixT) == 1 ? 0 : 1;
    if constexpr (P > kOnePassMax)
        return hipErrorInvalidValue;
    else if constexpr (P >= split_min(dtype))
        return launch_split_pack<P, PixT, CAP>(runs, count, stream);
    else
        return launch_reg_pack<P, PixT, CAP>(runs, count, stream);
}

template <typename PixT, int CAP>
hipError_t launch_reg_p(int p, const RegRun* runs, int count, hipStream_t stream) {
    switch (p) {
        case 0: return launch_one<0, PixT, CAP>(runs, count, stream);
        case 1: return launch_one<1, PixT, CAP>(runs, count, stream);
        case 2: return launch_one<2, PixT, CAP>(runs, count, stream);
        case 3: return launch_one<3, PixT, CAP>(runs, count, stream);
        case 4: return launch_one<4, PixT, CAP>(runs, count, stream);
        case 5: return launch_one<5, PixT, CAP>(runs, count, stream);
        case 6: return launch_one<6, PixT, CAP>(runs, count, stream);
        case 7: return launch_one<7, PixT, CAP>(runs, count, stream);
        case 8: return launch_one<8, PixT, CAP>(runs, count, stream);
        default: return hipErrorInvalidValue;
    }
}

template <typename PixT>
hipError_t launch_reg_any(int p, const RegRun* runs, int count, hipStream_t stream) {
    return count == 1 ? launch_reg_p<PixT, 1>(p, runs, count, stream)
                      : launch_reg_p<PixT, kPack>(p, runs, count, stream);
}

}  // namespace

size_t fht_scratch_bytes(const Geometry& g, int dtype) {
    // (bands of 256 rows no longer use theirs; callers' sizes stay what they were)
    static_assert(kOnePassMax >= kRegMaxP, "counted wherever two passes use it");
    if (g.p <= kRegMaxP) return 0;
    // [h/128 sub-blocks][2 directions][128 shifts][W]: uint16 for 8-bit pixels
    // (a 128-row line sum is at most 128 * 255), int32 for 16-bit ones
    const size_t cell = dtype == 0 ? sizeof(uint16_t) : sizeof(int32_t);
    return (size_t)(g.h >> kRegMaxP) * 2 * (1u << kRegMaxP) * (size_t)g.W * cell;
}

hipError_t launch_fht_jobs(const FhtJobSpec* jobs, int count, hipStream_t stream) {
    // Register-kernel runs, launched in packs of equal (row-block height, pixel type).
    std::vector<RegRun> runs;
    runs.reserve(count);
    for (int q = 0; q < count; ++q) {
        const FhtJobSpec& J = jobs[q];
        const Geometry& g = J.g;
        RegRun r;
        r.img = J.img;
        r.dtype = J.dtype;
        r.w = g.w;
        r.W = g.W;
        r.out16 = J.tables.narrow ? J.tables.tab16 : nullptr;
        r.narrow = 0;
        r.grid_mode = J.grid_mode;
        if (g.p <= kOnePassMax) {
            r.p = g.p;
            r.blocks = g.k;
            r.to_table = 1;
            r.out = J.tables.wide;
            r.narrow = J.tables.narrow;
        } else {  // tall bands: 128-row sub-blocks first, then the coarse levels
            r.p = kRegMaxP;
            r.blocks = g.h >> kRegMaxP;
            r.to_table = 0;
            r.out = static_cast<int32_t*>(J.scratch);
        }
        // Only the register kernel's grid has a choice: elsewhere it must not keep
        // runs from sharing a launch.
        if (r.p >= split_min(r.dtype)) r.grid_mode = 0;
        runs.push_back(r);
    }
    for (int dtype = 0; dtype < 2; ++dtype) {
        for (int p = 0; p <= kOnePassMax; ++p) {
            for (int gm = 0; gm < 2; ++gm) {
            std::vector<RegRun> group;
            for (const RegRun& r : runs)
                if (r.dtype == dtype && r.p == p && r.grid_mode == gm) group.push_back(r);
            for (size_t q0 = 0; q0 < group.size(); q0 += kPack) {
                const int n = (int)std::min<size_t>(kPack, group.size() - q0);
                hipError_t e = dtype == 0 ? launch_reg_any<uint8_t>(p, group.data() + q0, n, stream)
                                          : launch_reg_any<uint16_t>(p, group.data() + q0, n, stream);
                if (e != hipSuccess) return e;
            }
            }
        }
    }
    // Coarse levels of the tall bands.
    std::vector<CombineJob> comb;
    for (int q = 0; q < count; ++q) {
        const Geometry& g = jobs[q].g;
        if (g.p <= kOnePassMax) continue;
        CombineJob c;
        c.sub = jobs[q].scratch;
        c.sub16 = jobs[q].dtype == 0;
        c.tables = jobs[q].tables.wide;
        c.tab16 = jobs[q].tables.tab16;
        c.narrow = jobs[q].tables.narrow;
        c.p = g.p;
        c.W = g.W;
        c.k = g.k;
        c.tiles_x = (g.W + 255) / 256;
        c.item0 = 0;
        comb.push_back(c);
    }
    for (int sh = 2; sh <= 3; ++sh) {  // bands of 512 and 1024 rows
      for (int s16 = 0; s16 < 2; ++s16) {
        std::vector<CombineJob> group;
        for (const CombineJob& c : comb)
            if (c.p - kRegMaxP == sh && c.sub16 == s16) group.push_back(c);
        for (size_t q0 = 0; q0 < group.size(); q0 += kPack) {
            CombinePack pk{};
            const int n = (int)std::min<size_t>(kPack, group.size() - q0);
            long long total = 0;
            for (int q = 0; q < n; ++q) {
                pk.job[q] = group[q0 + q];
                pk.job[q].item0 = (int)total;
                total += (long long)pk.job[q].tiles_x * ((1LL << pk.job[q].p) / kShiftGroup) * 2 *
                         pk.job[q].k;
                if (total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
            }
            pk.count = n;
            pk.total = (int)total;
            TimedLaunch tl("fht_combine_kernel", stream);
            const dim3 grid((unsigned)total), block(256);
            if (s16) {
                if (sh == 2)
                    hipLaunchKernelGGL((fht_combine_kernel<2, uint16_t>), grid, block, 0, stream, pk);
                else
                    hipLaunchKernelGGL((fht_combine_kernel<3, uint16_t>), grid, block, 0, stream, pk);
            } else {
                if (sh == 2)
                    hipLaunchKernelGGL((fht_combine_kernel<2, int32_t>), grid, block, 0, stream, pk);
                else
                    hipLaunchKernelGGL((fht_combine_kernel<3, int32_t>), grid, block, 0, stream, pk);
            }
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
      }
    }
    return hipSuccess;
}

hipError_t launch_fht(const void* img, int dtype, const Geometry& g, const TableSet& tables,
                      void* scratch, hipStream_t stream, int grid_mode) {
    FhtJobSpec j{img, dtype, g, tables, scratch, grid_mode};
    return launch_fht_jobs(&j, 1, stream);
}

}  // namespace fhtp
