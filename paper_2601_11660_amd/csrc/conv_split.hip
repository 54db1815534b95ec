#include <type_traits>
#include "mbu_internal.h"
#include "mfma_common.h"

namespace mbu {

// Small layers: few pixels, many input channels (the deep levels of a 512 x 512 frame, every level of a
// smaller one).  The block kernel of conv_mfma.hip gives a wave 4 rows x 32 pixels x 64 channels and all
// input channels; such a layer then has fewer than 512 waves for 1024 SIMDs and its time is one wave's
// serial chain over the input steps.  Here the S waves of a block share one tile of R groups of 32 pixels
// (TWC columns x R * 32 / TWC rows) x 32 output channels and contract a slice of the input channels each;
// the partial sums (half-integers, exact in any order) meet in LDS.
//
// Every wave works alone until then: it fetches the weight fragments and the packed halo window of its
// slice, expands the window into LDS of its own, double buffered, a step ahead, as in the wave-private
// kernel of conv_mfma.hip.  Weights are refilled in place as soon as a fragment is free; a fetch beyond
// the slice gets an offset outside the buffer and moves nothing.  Narrow frames take tiles 8 or 16
// columns wide, whose 32 matrix columns are 4 or 2 image rows: a 4 x 6 frame is one group, not four.
//
// What bounds it: the tiny shapes by their latency chain (arguments, first fetch from beyond the L2, LDS,
// about 1.5 us next to the 2.5 us of a dispatch); 1024->1024 at 32 x 32 spends 12 K cycles in a block: 1.2 K
// issuing, 1.5 K for the first fetch, 4.6 K in the matrix loop (2 waves per SIMD: the matrix pipe is full),
// 4.2 K in the reduction, 0.7 K storing.  us per launch in a kernel trace, before -> now:
//   1024->1024 at 4x6 21.6 -> 5.2, at 32x32 22.3 -> 9.8;  512->1024 at 32x32 14.2 -> 6.5;
//   512->512 at 8x12 13.2 -> 4.2, at 64x64 14.1 -> 10.0;  256->512 at 64x64 9.1 -> 7.0;
//   256->256 at 16x24 8.7 -> 3.8;  128->128 at 32x48 7.3 -> 3.7;
//   [512 | 512]->512 at 64x64 24.2 -> 13.8
// (before: block kernel with four rows per wave; its two-row form stands at the rule below).  Up-sampled second inputs come here only where conv_upcat.hip does not take them.
// Measured and not kept: the whole window of all steps staged by the block in one go (coalesced, but a
// barrier and 2-3 dependent LDS passes before the first matrix instruction: 0.5-1 us slower on the tiny
// shapes, no faster on the others); 64 output channels per wave (no faster: the reduction doubles).
template <int R, int TWC>
struct SplitGeo {
    static constexpr int RS = 32 / TWC;              // image rows of a group
    static constexpr int TR = R * RS;                // image rows of the tile
    static constexpr int HR = TR + 2, HW = TWC + 2;  // halo window
    static constexpr int NPIX = HR * HW;
    static constexpr int NLD = (NPIX + 63) / 64;     // staged pixels per lane
    static constexpr int WIN = HR * 2 * HW;          // uint4 entries of a window, [row][half][col]
    static constexpr int PART = R * 4 * 64;          // float4 entries of a wave's accumulators
    static constexpr int WAVE = 2 * WIN > PART ? 2 * WIN : PART;   // LDS entries of a wave
    static constexpr int HEAD = 32 + R * 32;               // words: start values, output words
    static int lds_bytes(int s) { return HEAD * 4 + s * WAVE * 16; }
};

template <int R, int TWC, bool EVEN, bool TWO>
__global__ __launch_bounds__(512) void conv_mfma_split_kernel(
    const uint32_t *__restrict__ act, const uint32_t *__restrict__ low, int N, int H, int W, int Cwa, int Cwb,
    int low_shift, int Hb, int Wb, int ksteps, const uint4 *__restrict__ wfrag, int Cout, int log_s, int tiles_y,
    const int32_t *__restrict__ thresh, const int32_t *__restrict__ wsum,
    uint32_t *__restrict__ out_bits, uint32_t *__restrict__ out_pool)
{
    using G = SplitGeo<R, TWC>;
    constexpr int RS = G::RS, HW = G::HW, NLD = G::NLD;
    extern __shared__ uint4 lds[];
    const int S = 1 << log_s;
    float *start = reinterpret_cast<float *>(lds);
    uint32_t *words = reinterpret_cast<uint32_t *>(start + 32);
    uint4 *const body = lds + G::HEAD / 4;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    // channel tile fastest: consecutive blocks go to different XCDs, so where there are eight tiles or
    // more an XCD's L2 only sees its share of the weights.  A grid of three dimensions and slices by
    // shift: every division by an argument is 0.1 us of a latency chain of about 1.5.
    const int ct = blockIdx.x;
    int n = 0, ty = blockIdx.z;
    if (ty >= tiles_y) {
        n = ty / tiles_y;
        ty -= n * tiles_y;
    }
    const int y0 = ty * G::TR, x0 = (int)blockIdx.y * TWC;

    const int k_first = ksteps * wave >> log_s, k_end = ksteps * (wave + 1) >> log_s;
    const int Cw = Cwa + (TWO ? Cwb : 0);

    // ---- weights: fragments of the 32-channel tile, [tile64][kstep][tap][m][lane]
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(wfrag + ((size_t)(ct >> 1) * ksteps * 18 + (ct & 1)) * 64), 0, (ksteps * 18 - (ct & 1)) * 1024,
        0x00020000);
    constexpr uint32_t NOWHERE = 0x7ffffff0u;   // lane offset outside every buffer: reads 0, no traffic
    v4i Wg[3][3];   // [kx][ky]
    auto load_w = [&](uint32_t lane_off, int ks, int kx, int ky) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b128(wrs, lane_off, (ks * 18 + (ky * 3 + kx) * 2) * 1024, 0);
        Wg[kx][ky] = (v4i){(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
    };
    const uint32_t wlane = lane * 16;
#pragma unroll
    for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) load_w(wlane, k_first, kx, ky);

    // ---- staging plan: halo pixels lane + 64 * j
    uint4 *const win = body + wave * G::WAVE;
    const __amdgpu_buffer_rsrc_t ars =
        __builtin_amdgcn_make_buffer_rsrc((void *)act, 0, (int)((size_t)N * H * W * Cwa * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(TWO ? low : act), 0, TWO ? (int)((size_t)N * Hb * Wb * Cwb * 4) : 0, 0x00020000);
    uint32_t offa[NLD], offb[TWO ? NLD : 1];
    uint32_t inside = 0, inside_b = 0;
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
        int p = lane + 64 * j;
        p = p < G::NPIX ? p : 0;     // surplus lanes duplicate pixel 0 (same data, same slot)
        const int r = p / HW, c = p - r * HW;
        const int yy = y0 + r - 1, xx = x0 + c - 1;
        const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
        const int yc = min(max(yy, 0), H - 1), xc = min(max(xx, 0), W - 1);
        offa[j] = (uint32_t)((((size_t)n * H + yc) * W + xc) * Cwa * 4);
        inside |= (in ? 1u : 0u) << j;
        if (TWO) {
            const int yb = yc >> low_shift, xb = xc >> low_shift;
            inside_b |= ((in && yb < Hb && xb < Wb) ? 1u : 0u) << j;
            offb[j] = (uint32_t)((((size_t)n * Hb + min(yb, Hb - 1)) * Wb + min(xb, Wb - 1)) * Cwb * 4);
        }
    }
    uint2 gq[NLD];
    auto fetch = [&](int ks, bool want) {
        const int k0 = 2 * ks;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            if (EVEN) {   // both sources have an even word count: one aligned 8-byte load
                const bool b = TWO && k0 >= Cwa;
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(
                    b ? brs : ars, want ? (b ? offb[TWO ? j : 0] : offa[j]) : NOWHERE, (b ? k0 - Cwa : k0) * 4, 0);
                gq[j] = make_uint2(v[0], v[1]);
            } else {
                const int k1 = min(k0 + 1, Cw - 1);
                const bool b0 = TWO && k0 >= Cwa, b1 = TWO && k1 >= Cwa;
                gq[j].x = __builtin_amdgcn_raw_buffer_load_b32(
                    b0 ? brs : ars, want ? (b0 ? offb[TWO ? j : 0] : offa[j]) : NOWHERE, (b0 ? k0 - Cwa : k0) * 4, 0);
                gq[j].y = __builtin_amdgcn_raw_buffer_load_b32(
                    b1 ? brs : ars, want ? (b1 ? offb[TWO ? j : 0] : offa[j]) : NOWHERE, (b1 ? k1 - Cwa : k1) * 4, 0);
            }
        }
    };
    // word i & 1 of staged pixel i >> 1 of step ks (a word beyond the last meets zero weights)
    auto commit = [&](int ks, uint4 *buf, int i) {
        const int j = i >> 1;
        int p = lane + 64 * j;
        p = p < G::NPIX ? p : 0;
        const int r = p / HW, c = p - r * HW;
        const bool in = ((TWO && 2 * ks + (i & 1) >= Cwa ? inside_b : inside) >> j) & 1u;
        buf[(r * 2 + (i & 1)) * HW + c] =
            expand_word_masked((i & 1) ? gq[j].y : gq[j].x, in ? 0x22222222u : 0u, in ? 0u : 0x11111111u);
    };
    fetch(k_first, true);
    if (tid < 32) start[tid] = start_value(thresh[ct * 32 + tid], wsum[ct * 32 + tid]);
    for (int i = tid; i < R * 32; i += 64 * S) words[i] = 0;
#pragma unroll
    for (int i = 0; i < 2 * NLD; ++i) commit(k_first, win, i);

    v16f acc[R];
    const int tb_off = (col / TWC * 2 + half) * HW + col % TWC;
    constexpr int NROW = RS * (R - 1) + 3;    // first rows of the fragments of a tap column
    constexpr int NF = 3 * NROW;
    constexpr int NB = 3;
    // one input step; the first opens the accumulators
    auto step = [&](auto first, int ks) {
        const uint32_t wl = ks + 1 < k_end ? wlane : NOWHERE;
        const uint4 *tb = win + ((ks - k_first) & 1) * G::WIN + tb_off;
        uint4 *const nxt = win + ((ks - k_first + 1) & 1) * G::WIN;
        fetch(ks + 1, ks + 1 < k_end);
        __builtin_amdgcn_sched_barrier(0);
        v4i fr[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const uint4 b = tb[(j / NROW) + (j % NROW) * 2 * HW];
            fr[j] = (v4i){(int)b.x, (int)b.y, (int)b.z, (int)b.w};
        }
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int kx = j / NROW, rho = j % NROW;
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                const int d = rho - ky;
                if (d >= 0 && d % RS == 0 && d / RS < R) {
                    const bool opens = decltype(first)::value && kx == 0 && ky == 0;
                    acc[d / RS] = mfma_f4(Wg[kx][ky], fr[j % NB], opens ? (v16f)(0.0f) : acc[d / RS]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (j + NB < NF) {
                const int jn = j + NB;
                const uint4 b = tb[(jn / NROW) + (jn % NROW) * 2 * HW];
                fr[j % NB] = (v4i){(int)b.x, (int)b.y, (int)b.z, (int)b.w};
            }
            // fragment (kx, ky) is free after window row RS * (R - 1) + ky: refill for the next step
            if (rho >= RS * (R - 1)) load_w(wl, ks + 1, kx, rho - RS * (R - 1));
            if (j >= NF - 2 * NLD) commit(ks + 1, nxt, j - (NF - 2 * NLD));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    step(std::true_type{}, k_first);
    for (int ks = k_first + 1; ks < k_end; ++ks) step(std::false_type{}, ks);

    // ---- sum over the slices.  The partial sums take the place of the wave's windows (LDS instructions
    // of one wave execute in order); every unit of work is four channels of one group's pixels.
    float4 *const part = reinterpret_cast<float4 *>(win);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            part[(r * 4 + q) * 64 + lane] =
                make_float4(acc[r][4 * q], acc[r][4 * q + 1], acc[r][4 * q + 2], acc[r][4 * q + 3]);
    __syncthreads();
    const float4 *const sums = reinterpret_cast<const float4 *>(body);
    if (log_s == 3) reduce_slices<8, R>(sums, G::WAVE, start, words, wave, lane);
    else if (log_s == 2) reduce_slices<4, R>(sums, G::WAVE, start, words, wave, lane);
    else if (log_s == 1) reduce_slices<2, R>(sums, G::WAVE, start, words, wave, lane);
    else reduce_slices<1, R>(sums, G::WAVE, start, words, wave, lane);
    __syncthreads();
    const int Cow = Cout >> 5;
    if (out_bits)
        for (int i = tid; i < R * 32; i += 64 * S) {
            const int y = y0 + i / TWC, x = x0 + i % TWC;
            if (y < H && x < W) out_bits[(((size_t)n * H + y) * W + x) * Cow + ct] = words[i];
        }
    if (G::TR % 2 == 0 && out_pool) {
        // the tile origin is even: every 2x2 window lies inside the tile
        const int Hl = H >> 1, Wl = W >> 1;
        for (int i = tid; i < R * 8; i += 64 * S) {
            const int r = i / (TWC / 2), c = i % (TWC / 2);
            const int y = (y0 >> 1) + r, x = (x0 >> 1) + c;
            const uint32_t *p = words + 2 * r * TWC + 2 * c;
            if (y < Hl && x < Wl)
                out_pool[(((size_t)n * Hl + y) * Wl + x) * Cow + ct] = p[0] | p[1] | p[TWC] | p[TWC + 1];
        }
    }
}


// When, and with which tile.  Both sides measured with a kernel trace, caches flushed between launches; a unit
// is 9 matrix instructions (one group, 32 channels, one step):
//  - The block kernel with two rows per wave takes about 4.3 us + 0.8 per input step while its blocks have a
//    compute unit each; this kernel's time grows with groups x channel tiles, what its tiles cover beyond the
//    frame included.  They meet at 2048 of these, two for a SIMD.  Block -> here: 4 steps 53x128, 1792, 7.2 ->
//    6.2 us; 64x64, 2048, 7.0 -> 6.8; 192x96, 2304, 7.3 -> 7.2; 135x160, 2720, 7.2 -> 8.0.  8 steps 81x32, 1344,
//    10.2 -> 7.2; 64x64, 2048, 10.1 -> 8.5; 111x96, 2688, 10.4 -> 11.7.  16 steps 32x32, 1024, 16.8 -> 8.3; 64x128,
//    2048, 16.1 -> 14.1; 96x48, 2304, 16.5 -> 16.8.  Back to back with warm caches, 3 to 16 steps: 0.74-1.04 of
//    the block kernel's time at 1400 to 2048; 112x24, 256->768, 2688 of which 2016 in the frame, 6.1 us with the block
//    kernel, 7.4 here.  With two steps at 1792: 0.91 at 1500, 0.95 at 1750, 1.01 at 2000 with flushed caches, 1.05, 1.05
//    and 1.06 with warm ones.
//  - Tile: up to 4096 units a wave
//    takes a single group (every fragment is used once, but all waves run at once: [256 | 512 up]->256 at
//    16x24, 1152 units, 4.8 us against 5.6 with two groups); up to 12288 two groups
//    (512->1024 at 32x32, 8192 units, 6.5 us against 7.1 with one and 7.4 with four); then four, which
//    halve the weight traffic again (1024->1024 at 32x32, 16384 units, 9.8 against 10.5 us), as long as the
//    blocks of four slices are resident at once, two on a compute unit (1024->512 at 42x96, 528 blocks, 17.7 us
//    against 15.9 with two groups): up to the same line.
//    Tiles 32 wide only where they leave little more of the frame's width empty than tiles 16 wide, and a
//    frame of 8 columns or fewer stays with single groups 8 wide.
//  - One input step: nothing to split, but tiles of one group still spread a small layer further than the
//    row-streaming kernel's strips (64->64 at 64x64 4.3 against 5.4 us, 128x128, 1024 units, 4.8 against
//    5.3; even from 1200 units on, 64->128 at 128x128, 2048 units, 5.6 against 5.2).
//    Two inputs go to the block kernel otherwise, and are taken up to the line ([32 | 32]->64 at 75x131, 5.8 ->
//    4.2 us, [32 | 32]->32 at 151x263 5.4 -> 4.7).
//  - An up-sampled second input comes here where conv_upcat.hip does not take the layer (odd frames, skips
//    that are not a multiple of 64 channels, no summed taps), with any number of steps: [32 | 64]->32 at 64x96
//    6.9 -> 3.8 us, [64 | 128]->64 at 75x131 6.8 -> 4.8, [96 | 192]->96 at 64x96 8.2 -> 6.0, at 101x151, 1482,
//    8.5 -> 7.7, [128 | 256]->128 at 101x151, 1976, 9.0 -> 8.7.
//  - Slices: as many as give 2048 waves (two per SIMD), at most 8 and at most one per step.  Eight slices of
//    four groups take 129 KiB of LDS, one block on a compute unit: four, where there are more blocks than units
//    (512->128 at 106x128, 432 blocks, 11.0 -> 8.8 us).
SplitPlan conv_split_plan(int N, int H, int W, const BlobLayout &L, bool two, bool pool)
{
    SplitPlan p{0, 0, 0};
    const long ctiles = L.cout >> 5;
    if ((double)N * H * W * L.cin_words * 4 >= 1073741824.0) return p;
    long best = 0;
    for (int tw : {32, 16, 8}) {   // fewest groups; the widest of equals
        if (tw == 32 && pool) continue;   // a single row
        const long g = (long)N * ceil_div(W, tw) * ceil_div(H, 32 / tw);
        if (!p.tw || g < best) { p.tw = tw; best = g; }
    }
    const long units = best * ctiles * L.ksteps;
    if (L.ksteps == 1 && !two && units > 1200) return SplitPlan{0, 0, 0};
    p.r = 1;
    if (units > 4096 && W > 8) {
        p.r = 2;
        p.tw = 16;
        if (units > 12288 && 7 * round_up(W, 32) <= 8 * round_up(W, 16) &&
            (long)N * ceil_div(W, 32) * ceil_div(H, 4) * ctiles <= 512) { p.r = 4; p.tw = 32; }
    }
    const long tiles = (long)N * ceil_div(W, p.tw) * ceil_div(H, p.r * 32 / p.tw) * ctiles;
    if (tiles * p.r > (L.ksteps <= 2 ? 1792 : 2048)) return SplitPlan{0, 0, 0};
    const int most = p.r == 4 && tiles > 256 ? 2 : 3;
    p.log_s = 0;
    while (p.log_s < most && 2 << p.log_s <= L.ksteps && tiles << p.log_s < 2048) ++p.log_s;
    // the grid's second and third dimension end at 65535
    if (ceil_div(W, p.tw) > 65535 || (long)N * ceil_div(H, p.r * 32 / p.tw) > 65535) return SplitPlan{0, 0, 0};
    return p;
}

template <int R, int TWC>
static int launch_split_t(const SplitPlan &p, const uint32_t *act, int cwa, const uint32_t *low, int cwb, int low_shift,
                          int hb, int wb, int N, int H, int W, const BlobLayout &L, const void *blob,
                          const int32_t *thresh, uint32_t *out_bits, uint32_t *out_pool, hipStream_t s)
{
    using G = SplitGeo<R, TWC>;
    const uint4 *wfrag = (const uint4 *)((const uint8_t *)blob + L.off_f4);
    const int32_t *wsum = (const int32_t *)((const uint8_t *)blob + L.off_cnt) + (size_t)10 * L.cout_pad64;
    const int tiles_x = ceil_div(W, TWC), tiles_y = ceil_div(H, G::TR);
    const dim3 grid((unsigned)(L.cout >> 5), (unsigned)tiles_x, (unsigned)(N * tiles_y)), block(64 << p.log_s);
    const size_t shmem = G::lds_bytes(1 << p.log_s);
    const bool even = cwa % 2 == 0 && (!low || cwb % 2 == 0);
#define MBU_SPLIT(EVEN_, TWO_)                                                                                       \
    MBU_LAUNCH((conv_mfma_split_kernel<R, TWC, EVEN_, TWO_>), grid, block, shmem, s, act, low, N, H, W, cwa, cwb,     \
               low_shift, hb, wb, L.ksteps, wfrag, L.cout, p.log_s, tiles_y, thresh, wsum, out_bits, out_pool)
    if (low) {
        if (even) MBU_SPLIT(true, true);
        else MBU_SPLIT(false, true);
    } else {
        if (even) MBU_SPLIT(true, false);
        else MBU_SPLIT(false, false);
    }
#undef MBU_SPLIT
    return check_launch("conv_mfma_split");
}

int launch_conv_mfma_split(const SplitPlan &p, const uint32_t *act, int cwa, const uint32_t *low, int cwb,
                           int low_shift, int hb, int wb, int N, int H, int W, const BlobLayout &L, const void *blob,
                           const int32_t *thresh, uint32_t *out_bits, uint32_t *out_pool, hipStream_t s)
{
#define MBU_GO(R_, TW_)                                                                                             \
    if (p.r == R_ && p.tw == TW_)                                                                                   \
        return launch_split_t<R_, TW_>(p, act, cwa, low, cwb, low_shift, hb, wb, N, H, W, L, blob, thresh, out_bits, \
                                       out_pool, s)
    MBU_GO(4, 32);
    MBU_GO(2, 16);
    MBU_GO(1, 32);
    MBU_GO(1, 16);
    MBU_GO(1, 8);
#undef MBU_GO
    return fail(MBU_ERR_ARG, "conv_mfma_split: no such tile");
}

}  // namespace mbu
