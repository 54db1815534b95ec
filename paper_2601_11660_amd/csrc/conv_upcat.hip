// Masked-binary 3x3 convolution over [skip | 2x nearest up-sampled low] (Sec. 2.1: the decoder
// concatenates encoder features with the up-sampled decoder features), with the up-sampled
// part contracted at LOW resolution.
//
// Output pixel (2Y + dy, 2X + dx) sees the up-sampled image through its 3x3 window, but the
// nine taps fall on only 2 x 2 low-resolution pixels: rows {Y - 1, Y, Y} for dy = 0 and
// {Y, Y, Y + 1} for dy = 1, columns alike.  Summing the weights of the taps that share a low
// pixel gives, per parity class (dy, dx), a 2x2 kernel with entries in -4 .. 4 over the low
// tensor; zero padding of the up-sampled image is zero padding of the low tensor.  The FP4
// format (E2M1) holds 0, 1, 2, 3, 4 exactly, products and sums stay exact integers in fp32,
// so the result is bit-identical to the layer on the materialised tensor while the up-sampled
// channels cost 4 instead of 9 matrix instructions per step: with twice as many low channels
// as skip channels, 17/27 of the work.
//
// The four waves of a block are the four parity classes of the same 4 x 32 low pixels
// (8 x 64 output pixels) and 64 output channels: a wave's 32 matrix columns are output pixels
// of one class, i.e. every second pixel of every second row, and its accumulator tile is
// 4 rows x 32 columns x 64 channels as in the other kernels.  Per 64-channel step of the skip
// tensor the block stages a 10 x 66 pixel window, columns split by parity so that a wave's
// stride-2 fragments are contiguous in LDS; per 128 channels of the low tensor (two steps: a
// low step is only 32 matrix instructions per wave, too few per barrier) a 6 x 34 window.
// Everything else - FP4 codes, 0 / 1 activations and the start value that goes with them (a low
// pixel outside the image is 0.5 like any other), fragments rotating through three registers,
// fetches a step ahead through buffer resources, persistent blocks - is as in conv_mfma.hip.
//
// The window of the NEXT unit is fetched into registers at the start of a unit and expanded and
// written to the other LDS buffer one word per slot between the matrix instructions of the
// unit's later fragments: vector work hides only behind matrix instructions of the same wave.
// The slots are chosen so that every wait is a compile-time count (the staged words are older
// than the weight fragments fetched in the slots before) and the unit bodies are instantiated
// per kind of the next unit, so that no slot contains a branch: with a run-time branch in the
// slots the compiler drains the vector-memory counter there and the kernel gets slower, not
// faster (measured: 47.2 -> 49.9 us with branches, 47.2 -> 44.3 us without, 1536 -> 512).
#include "mbu_internal.h"
#include "mfma_common.h"
#include <algorithm>
#include <type_traits>

namespace mbu {

constexpr int UC_A_COLS = 66;                 // skip window: 66 pixels a row, 33 per column parity
constexpr int UC_A_ROW = 2 * 2 * 33;          // uint4 per window row: [half][parity][33]
constexpr int UC_B_COLS = 34;                 // low window
constexpr int UC_B_ROW = 2 * 34;              // uint4 per window row: [half][34]

// RW: low rows per block tile = output rows per wave
template <int RW>
__device__ __forceinline__ void upcat_layer(
    const uint32_t *__restrict__ act, const uint32_t *__restrict__ low, int N, int H, int W, int ksA,
    int ksL, const uint4 *__restrict__ wfrag, const uint4 *__restrict__ wup, int Cout, int tiles64,
    int ptiles, TileStep tstep, const int32_t *__restrict__ thresh, const int32_t *__restrict__ wsum,
    uint32_t *__restrict__ out_bits)
{
    constexpr int UC_A_ROWS = 2 * RW + 2;       // skip window
    constexpr int UC_B_ROWS = RW + 2;           // low window
    constexpr int UC_B_SLICE = UC_B_ROWS * UC_B_ROW;   // one 64-channel slice of the low window
    constexpr int UC_TILE = UC_A_ROWS * UC_A_ROW;      // the larger of the two windows (two low slices: 816 for RW = 4)
    constexpr int NB = 3;                       // activation fragments in flight per wave
    constexpr int NLA = (UC_A_ROWS * UC_A_COLS + 255) / 256;   // skip pixels per thread: 3 for RW = 4, 2 for RW = 2
    static_assert((NLA == 2 || NLA == 3) && 2 * NLA <= 2 * RW + 1 && 2 * UC_B_SLICE <= UC_TILE, "slots and buffers");
    __shared__ uint4 tile[2][UC_TILE];
    __shared__ float4 init_tab[4][2][2][4];     // [wave][half][m][4 x 4 channels]: start values

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tid = threadIdx.x;
    const int dy = wave >> 1, dx = wave & 1;     // parity class of this wave
    const int col = lane & 31, half = lane >> 5;
    const int Hl = H >> 1, Wl = W >> 1;
    const int Cwa = 2 * ksA, Cwb = 2 * ksL;
    // units of work per tile: ksA steps of 64 skip channels, then ksL / 2 steps of 128 low channels
    // (a low step is only 4 taps: two of them per barrier)
    const int units = ksA + (ksL >> 1);
    const int ct = blockIdx.y;                   // 64-channel output tile of the block

    if (col < 8) {   // lanes (half, col < 8) write float4 number col of their half
        const int m = col >> 2, q = col & 3;
        const int cbase = ct * 64 + m * 32 + 16 * half + 4 * q;
        int4 t = make_int4(0, 0, 0, 0), u = make_int4(0, 0, 0, 0);
        if (cbase < Cout) {
            t = *reinterpret_cast<const int4 *>(thresh + cbase);
            u = *reinterpret_cast<const int4 *>(wsum + cbase);
        }
        init_tab[wave][half][m][q] = make_float4(start_value(t.x, u.x), start_value(t.y, u.y),
                                                 start_value(t.z, u.z), start_value(t.w, u.w));
    }

    const __amdgpu_buffer_rsrc_t ars =
        __builtin_amdgcn_make_buffer_rsrc((void *)act, 0, N * H * W * Cwa * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t brs =
        __builtin_amdgcn_make_buffer_rsrc((void *)low, 0, N * Hl * Wl * Cwb * 4, 0x00020000);
    // 3x3 fragments [tile64][64-channel step][tap][m][lane]; combined fragments
    // [tile64][64-channel step][class][a][b][m][lane] (steps count skip and low channels alike)
    const int steps = ksA + ksL;
    const __amdgpu_buffer_rsrc_t w3 = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(wfrag + (size_t)ct * steps * (18 * 64)), 0, steps * (18 * 1024), 0x00020000);
    const __amdgpu_buffer_rsrc_t wu = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(wup + (size_t)ct * steps * (32 * 64)), 0, steps * (32 * 1024), 0x00020000);
    const int wlane = lane * 16;

    // ---- staging plan.  Skip window: pixel p = tid + 256 j -> window row p / 66, column p % 66
    // (image pixel (2 Y0 - 1 + row, 2 X0 - 1 + column)), stored at [row][half][column parity]
    // [column / 2].  Low window: pixel tid -> row tid / 34, column tid % 34 (low pixel
    // (Y0 - 1 + row, X0 - 1 + column)), stored at [64-channel slice][row][half][column].
    // The LDS positions do not depend on the tile: two registers hold the four of them.
    uint32_t dst01, dst2b;
    {
        int d[NLA];
#pragma unroll
        for (int j = 0; j < NLA; ++j) {
            int p = tid + 256 * j;
            p = p < UC_A_ROWS * UC_A_COLS ? p : 0;      // surplus threads duplicate pixel 0
            const int r = p / UC_A_COLS, c = p - r * UC_A_COLS;
            d[j] = r * UC_A_ROW + (c & 1) * 33 + (c >> 1);
        }
        const int p = tid < UC_B_ROWS * UC_B_COLS ? tid : 0;
        const int r = p / UC_B_COLS, c = p - r * UC_B_COLS;
        dst01 = (uint32_t)d[0] | ((uint32_t)d[1] << 16);
        dst2b = (uint32_t)d[NLA - 1] | ((uint32_t)(r * UC_B_ROW + c) << 16);
    }
    uint32_t offa[NLA], offb;     // byte offsets of the (clamped) pixels
    uint32_t inside = 0;          // bits 0..2: skip pixels inside the image; bit 3: low pixel
    auto plan = [&](const TilePos &tp) {
        const int Y0 = tp.ty * RW, X0 = tp.tx * 32, n = tp.n;
        inside = 0;
#pragma unroll
        for (int j = 0; j < NLA; ++j) {
            int p = tid + 256 * j;
            p = p < UC_A_ROWS * UC_A_COLS ? p : 0;
            const int r = p / UC_A_COLS, c = p - r * UC_A_COLS;
            const int yy = 2 * Y0 - 1 + r, xx = 2 * X0 - 1 + c;
            const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
            const int yc = min(max(yy, 0), H - 1), xc = min(max(xx, 0), W - 1);
            offa[j] = (uint32_t)((((n * H + yc) * W + xc) * Cwa) * 4);
            inside |= (in ? 1u : 0u) << j;
        }
        {
            const int p = tid < UC_B_ROWS * UC_B_COLS ? tid : 0;
            const int r = p / UC_B_COLS, c = p - r * UC_B_COLS;
            const int yy = Y0 - 1 + r, xx = X0 - 1 + c;
            const bool in = yy >= 0 && yy < Hl && xx >= 0 && xx < Wl;
            const int yc = min(max(yy, 0), Hl - 1), xc = min(max(xx, 0), Wl - 1);
            offb = (uint32_t)((((n * Hl + yc) * Wl + xc) * Cwb) * 4);
            inside |= (in ? 1u : 0u) << 3;
        }
    };
    uint2 gq[NLA];
    auto stage_issue = [&](int u) {
        if (u < ksA) {
#pragma unroll
            for (int j = 0; j < NLA; ++j) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(ars, offa[j], u * 8, 0);
                gq[j] = make_uint2(v[0], v[1]);
            }
        } else {   // four words: two 64-channel slices
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(brs, offb, (u - ksA) * 16, 0);
            gq[0] = make_uint2(v[0], v[1]);
            gq[1] = make_uint2(v[2], v[3]);
        }
    };
    auto expand_store = [&](uint2 g, bool in, uint4 *d0, uint4 *d1) {
        const uint32_t m2 = in ? 0x22222222u : 0u, p1 = in ? 0u : 0x11111111u;
        *d0 = expand_word_masked(g.x, m2, p1);
        *d1 = expand_word_masked(g.y, m2, p1);
    };
    auto stage_commit = [&](int u, uint4 *buf) {
        if (u < ksA) {
#pragma unroll
            for (int j = 0; j < NLA; ++j) {
                const uint32_t at = j == 0 ? (dst01 & 0xffffu) : j == 1 ? (dst01 >> 16) : (dst2b & 0xffffu);
                expand_store(gq[j], (inside >> j) & 1u, buf + at, buf + at + 2 * 33);
            }
        } else {
            const uint32_t at = dst2b >> 16;
#pragma unroll
            for (int q = 0; q < 2; ++q)
                expand_store(gq[q], (inside >> 3) & 1u, buf + q * UC_B_SLICE + at, buf + q * UC_B_SLICE + at + 34);
        }
    };

    // One word of that commit: the staged words of the next unit are expanded and written one per
    // slot between the matrix instructions of the current unit (vector work hides only behind
    // matrix instructions of the same wave).  SKIP: the next unit is a skip step (six words:
    // word i & 1 of staged pixel i >> 1), else a low unit (four words: word i & 1 of slice
    // i >> 1).  Everything but the data is a compile-time constant: no branches in the slots.
    auto commit_word = [&](auto SKIP, uint4 *buf, int i) {
        if constexpr (decltype(SKIP)::value) {
            const int j = i >> 1;
            const uint32_t at = (j == 0 ? (dst01 & 0xffffu) : j == 1 ? (dst01 >> 16) : (dst2b & 0xffffu)) + (i & 1) * (2 * 33);
            const bool in = (inside >> j) & 1u;
            buf[at] = expand_word_masked((i & 1) ? gq[j].y : gq[j].x, in ? 0x22222222u : 0u, in ? 0u : 0x11111111u);
        } else if (i < 4) {
            const int q = i >> 1;
            const uint32_t at = q * UC_B_SLICE + (dst2b >> 16) + (i & 1) * 34;
            const bool in = (inside >> 3) & 1u;
            buf[at] = expand_word_masked((i & 1) ? gq[q].y : gq[q].x, in ? 0x22222222u : 0u, in ? 0u : 0x11111111u);
        }
    };

    // ---- weights of a unit in registers.  Skip step: Wg[kx][ky][m] = tap (ky, kx).  Low double
    // step: the combined taps (a, b) of this wave's class for slice 0 in slots (kx, ky) = (b, a),
    // for slice 1 in slots (2, a) [b = 0] and (a, 2) [b = 1]; slot (2, 2) is idle.
    v4i Wg[3][3][2];
    // One load instruction per fragment whatever the unit's kind: resource and offset are
    // selected with scalar instructions.
    auto load_w = [&](int u, int kx, int ky) {
        const bool up = u >= ksA;
        if (kx == 2 && ky == 2) {
            const int s3 = min(u, ksA - 1);     // idle in a low unit: loaded all the same
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const auto w = __builtin_amdgcn_raw_buffer_load_b128(w3, wlane, (s3 * 18 + 8 * 2 + m) * 1024, 0);
                Wg[2][2][m] = (v4i){(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
            }
            return;
        }
        const int q = (kx < 2 && ky < 2) ? 0 : 1;
        const int b = q == 0 ? kx : (kx == 2 ? 0 : 1);
        const int a = q == 0 ? ky : (kx == 2 ? ky : kx);
        const int sl = ksA + 2 * (u - ksA) + q;          // 64-channel step of the slice
        const __amdgpu_buffer_rsrc_t rs = up ? wu : w3;
        const int off = up ? (sl * 32 + ((wave * 2 + a) * 2 + b) * 2) * 1024 : (u * 18 + (ky * 3 + kx) * 2) * 1024;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b128(rs, wlane, off + m * 1024, 0);
            Wg[kx][ky][m] = (v4i){(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
        }
    };

    const int stride = gridDim.x;
    TilePos cur = tile_pos(blockIdx.x, tstep.tiles_x, tstep.tiles_y);
    plan(cur);
    stage_issue(0);
#pragma unroll
    for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) load_w(0, kx, ky);
    stage_commit(0, tile[0]);
    __syncthreads();

    // fragment addresses of this lane (uint4 units from the start of a window buffer): window
    // column 2 col + dx + kx lies in parity plane (dx + kx) & 1 at index col + (dx + kx) / 2
    const int baseX = dy * UC_A_ROW + half * 66 + (dx & 1) * 33 + col;                        // kx = 0; kx = 2: + 1
    const int baseY = dy * UC_A_ROW + half * 66 + ((dx + 1) & 1) * 33 + ((dx + 1) >> 1) + col;  // kx = 1
    const int baseB = dy * UC_B_ROW + half * 34 + dx + col;                                   // + b

    const int Cow = Cout >> 5;
    const int widx = ct * 2 + half;
    const uint32_t psel = half ? 0x07060302u : 0x05040100u;
    int buf = 0;
    for (int pt = blockIdx.x; pt < ptiles; pt += stride) {
        v16f acc[RW][2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 f = init_tab[wave][half][m][q];
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    acc[r][m][4 * q] = f.x; acc[r][m][4 * q + 1] = f.y;
                    acc[r][m][4 * q + 2] = f.z; acc[r][m][4 * q + 3] = f.w;
                }
            }

        // ---- skip steps: fragment (kx, t) is window row dy + t, t = 2 r + ky
        auto skip_step = [&](int u, auto NEXT_SKIP) {
            const int un = u + 1;                   // a skip step or the first low unit
            const uint4 *tb = tile[buf];
            stage_issue(un);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int NT = 2 * RW + 1, NF = 3 * NT;
            v4i fr[NB];
            auto frag = [&](int j) {
                const int kx = j / NT, t = j % NT;
                const uint4 b = tb[(kx == 1 ? baseY : baseX) + (kx == 2 ? 1 : 0) + t * UC_A_ROW];
                return (v4i){(int)b.x, (int)b.y, (int)b.z, (int)b.w};
            };
#pragma unroll
            for (int j = 0; j < NB; ++j) fr[j] = frag(j);
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const int kx = j / NT, t = j % NT;
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
                    const int r2 = t - ky;
                    if (r2 >= 0 && (r2 & 1) == 0 && r2 / 2 < RW) {
#pragma unroll
                        for (int m = 0; m < 2; ++m)
                            acc[r2 / 2][m] = mfma_f4(Wg[kx][ky][m], fr[j % NB], acc[r2 / 2][m]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (j + NB < NF) fr[j % NB] = frag(j + NB);
                // tap (ky, kx) is done after t = 2 (RW - 1) + ky
                if (t >= 2 * (RW - 1)) load_w(un, kx, t - 2 * (RW - 1));
                // the next unit's window (fetched at the start of this one): one word per slot of
                // the last tap column, before that column's weight fetches
                if (j >= 2 * NT && j < 2 * NT + 2 * NLA) commit_word(NEXT_SKIP, tile[buf ^ 1], j - 2 * NT);
                __builtin_amdgcn_sched_barrier(0);
            }
            buf ^= 1;
            __syncthreads();
        };
        for (int u = 0; u + 1 < ksA; ++u) skip_step(u, std::true_type{});
        skip_step(ksA - 1, std::false_type{});
        // ---- low units: fragment (q, b, t) is slice q, window row dy + t, t = r + a
        auto low_unit = [&](int u, auto LAST) {
            constexpr bool last = decltype(LAST)::value;
            const int un = last ? 0 : u + 1;        // a low unit, or the next tile's first skip step
            if (last) {
                TilePos nxt = cur;
                if (pt + stride < ptiles) nxt.advance(tstep);
                plan(nxt);
            }
            const uint4 *tb = tile[buf];
            stage_issue(un);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int NT = RW + 1, NF = 4 * NT;
            v4i fr[NB];
            auto frag = [&](int j) {
                const int q = j / (2 * NT), b = j / NT % 2, t = j % NT;
                const uint4 v = tb[q * UC_B_SLICE + baseB + b + t * UC_B_ROW];
                return (v4i){(int)v.x, (int)v.y, (int)v.z, (int)v.w};
            };
#pragma unroll
            for (int j = 0; j < NB; ++j) fr[j] = frag(j);
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const int q = j / (2 * NT), b = j / NT % 2, t = j % NT;
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const int r = t - a;
                    // slot of the combined tap (a, b) of slice q
                    const int kx = q == 0 ? b : (b == 0 ? 2 : a), ky = q == 0 ? a : (b == 0 ? a : 2);
                    if (r >= 0 && r < RW) {
#pragma unroll
                        for (int m = 0; m < 2; ++m) acc[r][m] = mfma_f4(Wg[kx][ky][m], fr[j % NB], acc[r][m]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (j + NB < NF) fr[j % NB] = frag(j + NB);
                // combined tap (a, b) is done after t = RW - 1 + a: its slot is refilled for the
                // next unit; the idle slot too when the next tile's skip step follows
                if (t >= RW - 1) {
                    const int a = t - (RW - 1);
                    load_w(un, q == 0 ? b : (b == 0 ? 2 : a), q == 0 ? a : (b == 0 ? a : 2));
                }
                if (j == 0 && last) load_w(un, 2, 2);
                // the next unit's window, one word per slot (the first slots of the second slice's columns)
                if (q == 1 && t < NLA) commit_word(LAST, tile[buf ^ 1], b * NLA + t);
                __builtin_amdgcn_sched_barrier(0);
            }
            buf ^= 1;
            __syncthreads();
        };
        for (int u = ksA; u + 1 < units; ++u) low_unit(u, std::false_type{});
        low_unit(units - 1, std::true_type{});

        // ---- epilogue: row r of the wave is output row 2 (Y0 + r) + dy, column col is output
        // column 2 (X0 + col) + dx
        const int n = cur.n;
        const int x = 2 * (cur.tx * 32 + col) + dx;
        const bool ok = x < W && widx < Cow;
        uint32_t sgn[RW][2];
#pragma unroll
        for (int i = 15; i >= 0; --i)
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    sgn[r][m] = __builtin_amdgcn_alignbit(i == 15 ? 0u : sgn[r][m],
                                                          __float_as_uint(acc[r][m][i]), 31);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const uint32_t word = finish_word64(sgn[r][0], sgn[r][1], psel);
            const int y = 2 * (cur.ty * RW + r) + dy;
            if (ok && y < H) out_bits[(((size_t)n * H + y) * W + x) * Cow + widx] = word;
        }
        cur.advance(tstep);
    }
}

// Four low rows per wave, and two (launch_conv_mfma_upcat).
#define MBU_UPCAT_KERNEL(NAME, RW)                                                                                   \
    __global__ __launch_bounds__(256, 2) void NAME(                                                                  \
        const uint32_t *__restrict__ act, const uint32_t *__restrict__ low, int N, int H, int W, int ksA, int ksL,    \
        const uint4 *__restrict__ wfrag, const uint4 *__restrict__ wup, int Cout, int tiles64, int ptiles,            \
        TileStep tstep, const int32_t *__restrict__ thresh, const int32_t *__restrict__ wsum,                         \
        uint32_t *__restrict__ out_bits)                                                                              \
    {                                                                                                                 \
        upcat_layer<RW>(act, low, N, H, W, ksA, ksL, wfrag, wup, Cout, tiles64, ptiles, tstep, thresh, wsum, out_bits); \
    }
MBU_UPCAT_KERNEL(conv_mfma_upcat_kernel, 4)
MBU_UPCAT_KERNEL(conv_mfma_upcat_rows2_kernel, 2)
#undef MBU_UPCAT_KERNEL

// ---------------------------------------------------------------------------------
// The same contraction for small layers (a 512 x 512 frame's two deepest decoder levels, every level of a
// smaller frame), where the kernel above has fewer waves than the chip has SIMDs and a wave's time is its
// serial chain over the input steps.  The S waves of a block share one tile - one group of 32 low pixels
// (TWC columns x 32 / TWC rows), NC parity classes, 32 output channels - and contract a slice of the input
// steps each; the partial sums (half-integers, exact in any order) meet in LDS.  A wave with all four classes
// stages the window once for them and uses a skip fragment of the weights four times (36 matrix instructions
// for 9 + 16 fragments of weights and window), at the price of one use per low fragment; a wave with one class
// spreads the fewest pixels over four times as many compute units, whose rate of weight fetches is
// then the bound.  Every wave stages for itself: fetch of the next step's window and weights during a
// step, expansion into the other of two LDS buffers in slots between the matrix instructions, bodies
// instantiated per kind of the current and the next step (no branch in a slot).  A fetch beyond the slice
// gets an offset outside the buffer and moves nothing.
template <int NC, int TWC>
struct UpSplitGeo {
    static constexpr int RS = 32 / TWC;                       // low rows of the group
    static constexpr int AR = 2 * RS + 2, AC = 2 * TWC + 2;   // skip window, columns split by parity
    static constexpr int AROW = 4 * (TWC + 1);                // uint4 of a window row: [half][parity][TWC + 1]
    static constexpr int BR = RS + 2, BC = TWC + 2;           // low window
    static constexpr int BROW = 2 * BC;                       // uint4 of a window row: [half][BC]
    static constexpr int NLA = (AR * AC + 63) / 64, NLB = (BR * BC + 63) / 64;
    static constexpr int WIN = AR * AROW;                     // the larger of the two windows
    static constexpr int PART = NC * 4 * 64;
    static constexpr int WAVE = 2 * WIN > PART ? 2 * WIN : PART;
    static constexpr int HEAD = 32 + NC * 32;                 // words: start values, output words
    static int lds_bytes(int s) { return HEAD * 4 + s * WAVE * 16; }
};

template <int NC, int TWC>
__global__ __launch_bounds__(512) void conv_mfma_upcat_split_kernel(
    const uint32_t *__restrict__ act, const uint32_t *__restrict__ low, int N, int H, int W, int ksA, int ksL,
    const uint4 *__restrict__ wfrag, const uint4 *__restrict__ wup, int Cout, int log_s, int tiles_y,
    const int32_t *__restrict__ thresh, const int32_t *__restrict__ wsum, uint32_t *__restrict__ out_bits)
{
    static_assert(NC == 1 || NC == 4, "one parity class or all of them");
    using G = UpSplitGeo<NC, TWC>;
    constexpr int NLA = G::NLA, NLB = G::NLB;
    constexpr uint32_t NOWHERE = 0x7ffffff0u;
    extern __shared__ uint4 lds[];
    float *start = reinterpret_cast<float *>(lds);
    uint32_t *words = reinterpret_cast<uint32_t *>(start + 32);   // [class][pixel]
    uint4 *const body = lds + G::HEAD / 4;
    const int S = 1 << log_s;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int ct = blockIdx.x;     // (three grid dimensions: no division by an argument)
    const int cls0 = NC == 1 ? blockIdx.y & 3 : 0;
    int n = 0, ty = blockIdx.z;
    if (ty >= tiles_y) {
        n = ty / tiles_y;
        ty -= n * tiles_y;
    }
    const int Y0 = ty * G::RS, X0 = (int)(NC == 1 ? blockIdx.y >> 2 : blockIdx.y) * TWC;
    const int Hl = H >> 1, Wl = W >> 1;
    const int ksteps = ksA + ksL;
    uint4 *const win = body + wave * G::WAVE;

    // slice of the step sequence [skip steps | low steps], by matrix instructions (9 and 4 per class)
    auto step_at = [&](int cost) {
        return cost <= 9 * ksA ? (cost + 8) / 9 : ksA + (cost - 9 * ksA + 3) / 4;
    };
    const int total = 9 * ksA + 4 * ksL;
    const int k_first = step_at(total * wave >> log_s), k_end = step_at(total * (wave + 1) >> log_s);

    // ---- weights
    const int m = ct & 1;
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(wfrag + (size_t)(ct >> 1) * ksteps * (18 * 64)), 0, ksteps * (18 * 1024), 0x00020000);
    const __amdgpu_buffer_rsrc_t urs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(wup + (size_t)(ct >> 1) * ksteps * (32 * 64)), 0, ksteps * (32 * 1024), 0x00020000);
    constexpr int NWL = 4 * NC, NW = NWL > 9 ? NWL : 9;
    v4i Wg[NW];   // skip step: [kx][ky]; low step: [class][a][b]
    auto load_w = [&](auto is_low, bool want, int ks, int i) {
        const uint32_t off = want ? lane * 16 : NOWHERE;
        const auto w = decltype(is_low)::value
                           ? __builtin_amdgcn_raw_buffer_load_b128(urs, off, (ks * 32 + (cls0 * 4 + i) * 2 + m) * 1024, 0)
                           : __builtin_amdgcn_raw_buffer_load_b128(
                                 wrs, off, (ks * 18 + ((i % 3) * 3 + i / 3) * 2 + m) * 1024, 0);
        Wg[i] = (v4i){(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
    };

    // ---- staging plans: pixels lane + 64 * j of either window (surplus lanes duplicate pixel 0)
    const __amdgpu_buffer_rsrc_t ars =
        __builtin_amdgcn_make_buffer_rsrc((void *)act, 0, (int)((size_t)N * H * W * ksA * 8), 0x00020000);
    const __amdgpu_buffer_rsrc_t brs =
        __builtin_amdgcn_make_buffer_rsrc((void *)low, 0, (int)((size_t)N * Hl * Wl * ksL * 8), 0x00020000);
    uint32_t offa[NLA], offb[NLB], in_a = 0, in_b = 0;
#pragma unroll
    for (int j = 0; j < NLA; ++j) {
        int p = lane + 64 * j;
        p = p < G::AR * G::AC ? p : 0;
        const int y = 2 * Y0 - 1 + p / G::AC, x = 2 * X0 - 1 + p % G::AC;
        in_a |= (y >= 0 && y < H && x >= 0 && x < W ? 1u : 0u) << j;
        offa[j] = (uint32_t)((((size_t)n * H + min(max(y, 0), H - 1)) * W + min(max(x, 0), W - 1)) * ksA * 8);
    }
#pragma unroll
    for (int j = 0; j < NLB; ++j) {
        int p = lane + 64 * j;
        p = p < G::BR * G::BC ? p : 0;
        const int y = Y0 - 1 + p / G::BC, x = X0 - 1 + p % G::BC;
        in_b |= (y >= 0 && y < Hl && x >= 0 && x < Wl ? 1u : 0u) << j;
        offb[j] = (uint32_t)((((size_t)n * Hl + min(max(y, 0), Hl - 1)) * Wl + min(max(x, 0), Wl - 1)) * ksL * 8);
    }
    uint2 gq[NLA];
    auto fetch = [&](auto is_low, bool want, int ks) {
        constexpr bool LOW = decltype(is_low)::value;
#pragma unroll
        for (int j = 0; j < (LOW ? NLB : NLA); ++j) {
            const auto v = LOW ? __builtin_amdgcn_raw_buffer_load_b64(brs, want ? offb[LOW ? j : 0] : NOWHERE, (ks - ksA) * 8, 0)
                               : __builtin_amdgcn_raw_buffer_load_b64(ars, want ? offa[j] : NOWHERE, ks * 8, 0);
            gq[j] = make_uint2(v[0], v[1]);
        }
    };
    auto commit = [&](auto is_low, uint4 *buf, int i) {   // word i & 1 of staged pixel i >> 1
        constexpr bool LOW = decltype(is_low)::value;
        const int j = i >> 1, h = i & 1;
        int p = lane + 64 * j;
        p = p < (LOW ? G::BR * G::BC : G::AR * G::AC) ? p : 0;
        const int r = p / (LOW ? G::BC : G::AC), c = p % (LOW ? G::BC : G::AC);
        const bool in = ((LOW ? in_b : in_a) >> j) & 1u;
        buf[LOW ? r * G::BROW + h * G::BC + c : r * G::AROW + (h * 2 + (c & 1)) * (TWC + 1) + (c >> 1)] =
            expand_word_masked(h ? gq[j].y : gq[j].x, in ? 0x22222222u : 0u, in ? 0u : 0x11111111u);
    };

    v16f acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[c][i] = 0.0f;

    // One step.  Slot j: window fragment j, at position (row j % n, column j / n) of the n x n positions the
    // classes' taps fall on; the matrix instructions that use it; then the refill of the weights of which this
    // was the last use, and, in the last slots, one word of the next step's window.
    constexpr int NB = 3;
    const int lr = col / TWC, lc = col % TWC;
    const int dy0 = cls0 >> 1, dx0 = cls0 & 1;
    auto step = [&](auto is_low, auto next_low, int ks, const uint4 *cur, uint4 *nxt) {
        constexpr bool LOW = decltype(is_low)::value, NLOW = decltype(next_low)::value;
        constexpr int K = LOW ? 2 : 3, P = K + (NC == 4 ? 1 : 0), NF = P * P;
        const bool more = ks + 1 < k_end;
        fetch(next_low, more, ks + 1);
        __builtin_amdgcn_sched_barrier(0);
        auto frag = [&](int j) {
            const int pr = j % P, pc = j / P;
            uint4 b;
            if (LOW) {
                b = cur[(lr + dy0 + pr) * G::BROW + half * G::BC + lc + dx0 + pc];
            } else {
                const int x = dx0 + pc;
                b = cur[(2 * lr + dy0 + pr) * G::AROW + (half * 2 + (x & 1)) * (TWC + 1) + lc + (x >> 1)];
            }
            return (v4i){(int)b.x, (int)b.y, (int)b.z, (int)b.w};
        };
        v4i fr[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) fr[j] = frag(j);
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int pr = j % P, pc = j / P;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int ky = pr - (c >> 1), kx = pc - (c & 1);
                if (ky >= 0 && ky < K && kx >= 0 && kx < K)
                    acc[c] = mfma_f4(Wg[LOW ? c * 4 + ky * 2 + kx : kx * 3 + ky], fr[j % NB], acc[c]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (j + NB < NF) fr[j % NB] = frag(j + NB);
            if (LOW) {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int ky = pr - (c >> 1), kx = pc - (c & 1);
                    if (ky >= 0 && ky < K && kx >= 0 && kx < K) load_w(next_low, more, ks + 1, c * 4 + ky * 2 + kx);
                }
            } else {
                const int ky = pr - (P - K), kx = pc - (P - K);
                if (ky >= 0 && kx >= 0) {
                    if (!NLOW || kx * 3 + ky < NWL) load_w(next_low, more, ks + 1, kx * 3 + ky);
                    if (NLOW && 9 + kx * 3 + ky < NWL) load_w(next_low, more, ks + 1, 9 + kx * 3 + ky);
                }
            }
            // the words of the next window over the last slots
            constexpr int NWORD = 2 * (NLOW ? NLB : NLA), PER = (NWORD + NF - 1) / NF, FROM = NF - (NWORD + PER - 1) / PER;
            if (j >= FROM)
#pragma unroll
                for (int i = (j - FROM) * PER; i < (j - FROM + 1) * PER && i < NWORD; ++i) commit(next_low, nxt, i);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::true_type LOW_STEP{};
    constexpr std::false_type SKIP_STEP{};
    if (k_first < k_end) {
        if (k_first < ksA) {
            fetch(SKIP_STEP, true, k_first);
#pragma unroll
            for (int i = 0; i < 9; ++i) load_w(SKIP_STEP, true, k_first, i);
#pragma unroll
            for (int i = 0; i < 2 * NLA; ++i) commit(SKIP_STEP, win, i);
        } else {
            fetch(LOW_STEP, true, k_first);
#pragma unroll
            for (int i = 0; i < NWL; ++i) load_w(LOW_STEP, true, k_first, i);
#pragma unroll
            for (int i = 0; i < 2 * NLB; ++i) commit(LOW_STEP, win, i);
        }
    }
    if (tid < 32) start[tid] = start_value(thresh[ct * 32 + tid], wsum[ct * 32 + tid]);
    for (int i = tid; i < NC * 32; i += 64 * S) words[i] = 0;
    auto cur = [&](int ks) { return win + ((ks - k_first) & 1) * G::WIN; };
    int ks = k_first;
    // skip steps that a skip step or nothing follows, the one before the first low step, low steps
    const int skips = k_end <= ksA ? k_end : ksA - 1;
    for (; ks < skips; ++ks) step(SKIP_STEP, SKIP_STEP, ks, cur(ks), cur(ks + 1));
    if (ks < ksA && ks < k_end) {
        step(SKIP_STEP, LOW_STEP, ks, cur(ks), cur(ks + 1));
        ++ks;
    }
    for (; ks < k_end; ++ks) step(LOW_STEP, LOW_STEP, ks, cur(ks), cur(ks + 1));

    // ---- sum over the slices, in the place of the wave's windows; a unit is four channels of one class
    float4 *const part = reinterpret_cast<float4 *>(win);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            part[(c * 4 + q) * 64 + lane] =
                make_float4(acc[c][4 * q], acc[c][4 * q + 1], acc[c][4 * q + 2], acc[c][4 * q + 3]);
    __syncthreads();
    const float4 *const sums = reinterpret_cast<const float4 *>(body);
    if (log_s == 3) reduce_slices<8, NC>(sums, G::WAVE, start, words, wave, lane);
    else if (log_s == 2) reduce_slices<4, NC>(sums, G::WAVE, start, words, wave, lane);
    else if (log_s == 1) reduce_slices<2, NC>(sums, G::WAVE, start, words, wave, lane);
    else reduce_slices<1, NC>(sums, G::WAVE, start, words, wave, lane);
    __syncthreads();
    const int Cow = Cout >> 5;
    for (int i = tid; i < NC * 32; i += 64 * S) {
        const int c = cls0 + (i >> 5), p = i & 31;
        const int y = 2 * (Y0 + p / TWC) + (c >> 1), x = 2 * (X0 + p % TWC) + (c & 1);
        if (y < H && x < W) out_bits[(((size_t)n * H + y) * W + x) * Cow + ct] = words[i];
    }
}

// Combined weights of the up-sampled channels.  Thread (o, class, a, b, word k) sums the taps
// of the 3x3 kernel that fall on low pixel (a, b) of class (dy, dx) for 32 input channels and
// stores the E2M1 codes of the sums as one
// 16-byte fragment: uint4 [cout_pad64/64][ksteps][class][a][b][2][64 lanes], nibble q of dword d
// = input channel 32k + 4q + d, lane = 32 (k & 1) + tile row of the output channel.
__global__ __launch_bounds__(256) void pack_upcat_kernel(const int8_t *__restrict__ w, BlobLayout L,
                                                         uint8_t *__restrict__ blob)
{
    const int words = 2 * L.ksteps;
    const long total = (long)L.cout_pad64 * 16 * words;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int k = (int)(idx % words);
    const int tab = (int)((idx / words) % 16);
    const int o = (int)(idx / (16L * words));
    const int cls = tab >> 2, a = (tab >> 1) & 1, b = tab & 1;
    const int dy = cls >> 1, dx = cls & 1;
    // rows of the 3x3 kernel on low row a: dy = 0: {0}, {1, 2};  dy = 1: {0, 1}, {2}
    const int ky0 = dy == 0 ? (a ? 1 : 0) : (a ? 2 : 0), ky1 = dy == 0 ? (a ? 2 : 0) : (a ? 2 : 1);
    const int kx0 = dx == 0 ? (b ? 1 : 0) : (b ? 2 : 0), kx1 = dx == 0 ? (b ? 2 : 0) : (b ? 2 : 1);
    uint32_t d[4] = {0, 0, 0, 0};
    if (o < L.cout && k < L.cin_words) {
        const int n = min(32, L.cin - k * 32);
        for (int i = 0; i < n; ++i) {
            int v = 0;
            for (int ky = ky0; ky <= ky1; ++ky)
                for (int kx = kx0; kx <= kx1; ++kx) v += w[((long)o * 9 + ky * 3 + kx) * L.cin + (long)k * 32 + i];
            const int mag = v < 0 ? -v : v;     // 0..4 -> E2M1 0, 1.0, 2.0, 3.0, 4.0
            const uint32_t code = (mag == 0 ? 0u : mag == 1 ? 2u : mag == 2 ? 4u : mag == 3 ? 5u : 6u) |
                                  (v < 0 ? 8u : 0u);
            d[i & 3] |= code << (4 * (i >> 2));
        }
    }
    const int tile64 = o >> 6, m = (o >> 5) & 1;
    const int row = tile_channel_to_row(o & 31);
    const int lane = (k & 1) * 32 + row;
    uint4 *F = reinterpret_cast<uint4 *>(blob + L.off_up);
    const size_t at = (((((size_t)tile64 * L.ksteps + (k >> 1)) * 4 + cls) * 4 + a * 2 + b) * 2 + m) * 64 + lane;
    F[at] = make_uint4(d[0], d[1], d[2], d[3]);
}

int launch_pack_upcat(const int8_t *w, const BlobLayout &L, void *blob, hipStream_t s)
{
    const long total = (long)L.cout_pad64 * 16 * 2 * L.ksteps;
    MBU_LAUNCH(pack_upcat_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, w, L, (uint8_t *)blob);
    return check_launch("pack_upcat_weights");
}

bool conv_upcat_supported(int Ca, int Clow, int N, int H, int W, const BlobLayout &L, const uint32_t *out_bits,
                          const uint32_t *out_pool)
{
    const double lim = 1073741824.0;   // byte offsets are computed in 32 bits
    return (L.sections & MBU_BLOB_SUMMED_TAPS) && out_bits && !out_pool && Ca > 0 && Clow > 0 && Ca % 64 == 0 && Clow % 128 == 0 && !(H & 1) && !(W & 1) &&
           (double)N * H * W * (Ca / 32) * 4 < lim && (double)N * (H / 2) * (W / 2) * (Clow / 32) * 4 < lim &&
           (double)L.ksteps * 32 * 1024 < lim;
}

// When, and with which tile (us in a kernel trace):
//  - The large kernel with two rows per wave takes 5.5 us with 3 input steps, 7.1 with 6, 10 with 12 and 16.5 with
//    24 while its blocks have a compute unit each; this one's time grows with tiles (a group of 32 low
//    pixels x 32 channels).  They meet at 384 tiles + 16 per step.  Large kernel -> here: [64 | 128]->64 at 128x192,
//    384 tiles, 5.7 -> 5.6, at 128x256, 512, 5.6 -> 6.2; [128 | 256]->128 at 96x128, 384, 7.0 -> 6.8, at 96x192, 576, 7.1 ->
//    8.2; [256 | 512]->256 at 64x128, 512, 9.8 -> 8.9, at 96x128, 768, 10.4 -> 11.4; [512 | 1024]->512 at 64x64, 512,
//    16.2 -> 13.2, at 64x96, 768, 16.8 -> 16.6, at 64x128, 1024, 16.8 -> 21.1.
//  - One class per wave up to 40000 matrix instructions in all ([512 | 1024]->512 at 8x12, 8704, 26.0 -> 6.0
//    against 8.3 with four; [64 | 128]->64 at 120x160, 20400, 6.5 against 7.7), four beyond
//    (81600, [128 | 256]->128 at 120x160, 10.6 against 11.6; 104448, 30x40, 24.9 -> 8.6 against 12.0).
//  - Fewest groups; of equals the narrow ones, whose window has fewer pixels.
//  - As many slices as stay within 2048 waves (two per SIMD), at most 8 and one per step.
struct UpSplitPlan {
    int nc, tw, log_s;   // nc = 0: the large kernel
};
static UpSplitPlan upcat_split_plan(int N, int Hl, int Wl, int ksA, int ksL, const BlobLayout &L)
{
    UpSplitPlan p{0, 0, 0};
    const int ksteps = ksA + ksL;
    const long g8 = (long)N * ceil_div(Wl, 8) * ceil_div(Hl, 4), g16 = (long)N * ceil_div(Wl, 16) * ceil_div(Hl, 2);
    p.tw = g8 <= g16 ? 8 : 16;
    // the grid's second and third dimension end at 65535
    if (4L * ceil_div(Wl, p.tw) > 65535 || (long)N * ceil_div(Hl, 32 / p.tw) > 65535) return p;
    const long tiles = std::min(g8, g16) * (L.cout >> 5);
    if (tiles > 384 + 16 * ksteps) return p;
    p.nc = tiles * (36 * ksA + 16 * ksL) <= 40000 ? 1 : 4;
    const long blocks = tiles * (4 / p.nc);
    while (p.log_s < 3 && 2 << p.log_s <= ksteps && blocks * 2 << p.log_s <= 2048) ++p.log_s;
    return p;
}

template <int NC, int TWC>
static int launch_upcat_split(int log_s, const uint32_t *act, int Ca, const uint32_t *low, int Clow, int N, int H, int W,
                              const BlobLayout &L, const uint4 *wfrag, const uint4 *wup, const int32_t *thresh,
                              const int32_t *wsum, uint32_t *out_bits, hipStream_t s)
{
    using G = UpSplitGeo<NC, TWC>;
    const int tiles_x = ceil_div(W / 2, TWC), tiles_y = ceil_div(H / 2, G::RS);
    MBU_LAUNCH((conv_mfma_upcat_split_kernel<NC, TWC>),
               dim3((unsigned)(L.cout >> 5), (unsigned)(tiles_x * (4 / NC)), (unsigned)(N * tiles_y)), dim3(64 << log_s),
               (size_t)G::lds_bytes(1 << log_s), s, act, low, N, H, W, Ca / 64, Clow / 64, wfrag, wup, L.cout, log_s,
               tiles_y, thresh, wsum, out_bits);
    return check_launch("conv_mfma_upcat_split");
}

int launch_conv_mfma_upcat(const uint32_t *act, int Ca, const uint32_t *low, int Clow, int N, int H, int W,
                           const BlobLayout &L, const void *blob, const int32_t *thresh, uint32_t *out_bits,
                           hipStream_t s)
{
    const uint4 *wfrag = (const uint4 *)((const uint8_t *)blob + L.off_f4);
    const uint4 *wup = (const uint4 *)((const uint8_t *)blob + L.off_up);
    // sums of the weights per output channel: row 10 of the count section
    const int32_t *wsum = (const int32_t *)((const uint8_t *)blob + L.off_cnt) + (size_t)10 * L.cout_pad64;
    if (t_cfg.tune_rw == 0) {
        const UpSplitPlan p = upcat_split_plan(N, H / 2, W / 2, Ca / 64, Clow / 64, L);
#define MBU_GO(NC_, TW_)                                                                                        \
    if (p.nc == NC_ && p.tw == TW_)                                                                             \
        return launch_upcat_split<NC_, TW_>(p.log_s, act, Ca, low, Clow, N, H, W, L, wfrag, wup, thresh, wsum, out_bits, s)
        MBU_GO(1, 8);
        MBU_GO(1, 16);
        MBU_GO(4, 8);
        MBU_GO(4, 16);
#undef MBU_GO
    }
    const int tiles64 = L.cout_pad64 / 64;
    // Two low rows per wave instead of four where the blocks of four leave compute units empty or with one block: while
    // those of two have a unit each ([64 | 128]->64 at 256x256, 128 -> 256 blocks, 7.8 -> 5.9 us; [128 | 256]->128 at
    // 128x256 10.6 -> 7.7; [256 | 512]->256 at 128x128 14.3 -> 10.1; [512 | 1024]->512 at 64x128 23.8 -> 16.8), and with few
    // input steps, whose weights then cost less than the second wave of a SIMD gains, while they have two (256 -> 512:
    // [64 | 128]->64 at 256x512 8.5 -> 7.8, [256 | 512]->256 at 128x256 15.2 -> 15.0, but [512 | 1024]->512 at 128x128 26.2 ->
    // 28.3).  Beyond, the weights are fetched twice as often for nothing ([256 | 512]->256 at 160x240 23.1 -> 25.1).
    // (Kernel trace with the caches flushed between launches; back to back on warm caches 6.6 -> 5.2, 9.1 -> 6.7, 13.9 ->
    // 9.7, 23.9 -> 17.7 and 6.7 -> 6.5, 14.8 -> 15.0.)
    const int tiles_x = ceil_div(W / 2, 32);
    const long blocks2 = (long)N * ceil_div(H / 2, 2) * tiles_x * tiles64;
    const int rw = t_cfg.tune_rw == 0 && blocks2 <= ((Ca + Clow) / 64 <= 12 ? 512 : 256) ? 2 : 4;
    const int tiles_y = ceil_div(H / 2, rw);
    const long tiles = (long)N * tiles_y * tiles_x;
    if (tiles > 0x7fffffffL) return fail(MBU_ERR_SHAPE, "too many tiles for one launch");
    // persistent blocks: two per compute unit in total, spread over the 64-channel tiles
    const int gx = (int)std::min(tiles, (long)std::max(1, 512 / tiles64));
    const TileStep tstep = tile_step(gx, tiles_x, tiles_y);
    const dim3 grid((unsigned)gx, (unsigned)tiles64), block(256);
    if (rw == 2)
        MBU_LAUNCH(conv_mfma_upcat_rows2_kernel, grid, block, 0, s, act, low, N, H, W, Ca / 64, Clow / 64, wfrag, wup, L.cout,
                   tiles64, (int)tiles, tstep, thresh, wsum, out_bits);
    else
        MBU_LAUNCH(conv_mfma_upcat_kernel, grid, block, 0, s, act, low, N, H, W, Ca / 64, Clow / 64, wfrag, wup, L.cout,
                   tiles64, (int)tiles, tstep, thresh, wsum, out_bits);
    return check_launch("conv_mfma_upcat");
}

}  // namespace mbu
