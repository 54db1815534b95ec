// Full-precision first layer (Sec. 4.1) on the matrix cores, with sign bits that are
// identical to those of the sequential float32 definition.
//
// Definition (what the output bits must equal): y = sum over (ky, kx, ci) in that order of
// w * x, started at 0.0f, one fused multiply-add per term, zero padding; bit = (y >= 0).
// Only the SIGN of y leaves this layer, and the sign of a sum is known without the exact
// rounding sequence whenever a cheaper estimate is further from zero than its own error:
//
//   scaling        the sign of y[o, p] does not change when the weights of output channel o and
//                  the patch of pixel p are each multiplied by a positive power of two, so
//                  every weight row and every patch is scaled (exactly) to a Euclidean norm
//                  in [2^12, 2^13): whatever the magnitudes of the inputs, fp16 then neither
//                  overflows (values < 2^13) nor loses more than 2^-25 absolute per value to
//                  its subnormal range (2^-37 of the norm; 2^-26 of it if subnormal inputs
//                  were flushed);
//   fast estimate  every scaled float is split into two fp16 terms v = vh + vl + r, both
//                  rounded to nearest, |r| <= 2^-22 |v|; yf = sum wh*xh + wh*xl + wl*xh on
//                  v_mfma_f32_32x32x16_f16 (fp16 products are exact in the fp32 accumulator);
//   error budget   |yf - y| <= kappa * ||w_o||_2 * ||x_patch||_2 (in scaled units), every term
//                  relative to S = sum |w||x| <= ||w||_2 ||x||_2 (see STEM_KAPPA below): the
//                  rounding of the sequential chain itself, the terms the split drops, and the
//                  additions inside the matrix instructions, bounded for ANY order of addition
//                  and for rounding to nearest or truncation to 24 bits alike;
//   decision       |yf| >  T = kappa * max_o ||w_o|| * ||x_patch||  ->  sign(y) = sign(yf);
//                  otherwise the output is recomputed by the sequential chain itself, on the
//                  unscaled float32 inputs.
//
// About 1 output in 10^5 takes the second route with normally distributed data, so the
// layer costs 12 matrix instructions per 32 pixels x 64 channels instead of 64 x 27 fused
// multiply-adds per pixel.  Non-finite inputs, and norms outside [2^-60, 2^60], make T
// infinite and send every affected output down the sequential route; an all-zero patch gives
// +0.0f without any arithmetic.
//
// GEMM view: D[channel][pixel] = sum_k Wt[channel][k] * X[k][pixel], k = (ky*3 + kx)*Ci + ci
// (the memory order of the weights), padded to KT*16.  A wave owns 64 output channels
// (two 32-row tiles, weights scaled and split once and kept in registers) and walks over
// tiles of 32 consecutive pixels of an image row.  Lane (column j, half h) gathers the patch
// values k = 16t + 8h + i of pixel x0 + j through a raw buffer resource - a border tap or a
// padded k gets an offset beyond the buffer and reads 0.0f.
#include "mbu_internal.h"
#include "mfma_common.h"
#include <algorithm>
#include <type_traits>

namespace mbu {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// Error budget of the fast estimate relative to S = sum |w_k||x_k| <= ||w||_2 ||x||_2, worst
// case, no measured term:
//   sequential chain (the definition's own rounding): 27 fused multiply-adds, each within 2^-24
//     of a partial sum that is at most S in magnitude                       27 * 2^-24 = 1.61e-6
//   terms the split drops: wl*xl, rw*x, w*rx with |wl|, |xl| <= 2^-11, |rw|, |rx| <= 2^-22
//     of the value                                                        ~  3 * 2^-22 = 0.72e-6
//   additions inside the matrix instructions.  The products of two fp16 values are exact in
//     fp32; what is assumed of the hardware is only that every addition it performs - in
//     whatever order - is accurate to 2^-23 of its result (round to nearest gives 2^-24,
//     truncation to 24 bits 2^-23).  The two groups of small products (wl*xh, wh*xl; at most
//     2^-10 S in total) are accumulated FIRST, while the accumulator is below 2^-10 S, so
//     their 56 additions contribute below 1e-8; the 28 additions of the wh*xh group (27 terms
//     and the constant) happen on partial sums of at most S(1 + 2^-9)        28 * 2^-23 = 3.34e-6
//   total 5.68e-6 < kappa = 2^-17 = 7.63e-6.
constexpr float STEM_KAPPA = 0x1p-17f;
constexpr uint32_t OOB = 0x80000000u;   // byte offset beyond any accepted image

// (a, b) -> packed fp16 pairs hi and lo with v = hi + lo + r, |r| <= 2^-22 |v| (+ 2^-25):
// both conversions round to nearest and the remainder is computed without error
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &hi, uint32_t &lo)
{
    const v2f f = {a, b};
    const v2h h = __builtin_convertvector(f, v2h);
    const v2f r = f - __builtin_convertvector(h, v2f);
    hi = __builtin_bit_cast(uint32_t, h);                                   // low half = a
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2h));
}

// the power of two that brings a norm in [2^-60, 2^60] into [2^12, 2^13)
__device__ __forceinline__ float norm_scale(float nrm)
{
    const uint32_t e = (__float_as_uint(nrm) >> 23) & 0xffu;               // nrm in [2^(e-127), 2^(e-126))
    return __uint_as_float((266u - e) << 23);                              // 2^(12 - (e - 127))
}

__device__ __forceinline__ v8h as_v8h(const uint4 &v) { return __builtin_bit_cast(v8h, v); }

__device__ __forceinline__ float swap_add(float v)
{
    const uint32_t u = __float_as_uint(v);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// whether the values of both lane halves are all +-0 (bits: OR of their bit patterns).  A norm of 0 does not say
// so: the squares of values below 2^-75 round to 0
__device__ __forceinline__ bool all_zero(uint32_t bits)
{
    const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
    return ((sw[0] | sw[1]) << 1) == 0;
}

template <int CI, bool WRITE_PRE>
__global__ __launch_bounds__(256) void stem_mfma_kernel(
    const float *__restrict__ img, uint32_t img_bytes, int N, int H, int W,
    const float *__restrict__ w, int Co, int nchunks, int nslots, int ntiles, TileStep tstep,
    uint32_t *__restrict__ out, float *__restrict__ pre)
{
    constexpr int KV = 9 * CI;             // terms per output
    constexpr int KT = (KV + 15) / 16;     // 16-wide K blocks
    constexpr int NS = KT * 8;             // patch values per lane
    // k = KV is the first padded term; it lives in slot BIAS_SLOT of the lanes of half BIAS_HALF
    constexpr int BIAS_SLOT = 8 * (KV / 16) + (KV % 8), BIAS_HALF = (KV / 8) % 2;
    static_assert(KV < 16 * KT, "a padded k is needed for the constant term");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gw = blockIdx.x * 4 + wave;
    if (gw >= nchunks * nslots) return;    // whole wave leaves; nothing is shared
    const int chunk = gw % nchunks;        // 64 output channels, fixed for the wave
    const int slot = gw / nchunks;
    const int col = lane & 31, half = lane >> 5;
    const bool tile1 = chunk * 64 + 32 < Co;   // second 32-channel tile exists (Co % 32 == 0)

    // ---- weights of this wave: every row scaled to a norm in [2^12, 2^13), split once, kept
    // in registers.  The lane holds half of the K range of row `col` of both channel tiles.
    uint4 Wh[2][KT], Wl[2][KT];
    float row_unscale[2];   // 1 / scale of this lane's row (exact), for the diagnostic output
    uint32_t rb = 0;        // bit pattern of the largest scaled row norm (see below)
    bool w_sane = true;     // every row norm is finite and inside [2^-60, 2^60], or exactly 0
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int ch = chunk * 64 + m * 32 + tile_row_to_channel(col);
        float v[NS];
        float part = 0.0f;
        uint32_t bits = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = 16 * (s >> 3) + 8 * half + (s & 7);
            const bool ok = ch < Co && k < KV;
            const float wv = w[ok ? (size_t)ch * KV + k : 0];   // unconditional load
            v[s] = ok ? wv : 0.0f;
            part = __builtin_fmaf(v[s], v[s], part);
            bits |= __float_as_uint(v[s]);
        }
        const float nrm = __builtin_sqrtf(swap_add(part));      // both halves: ||w_row||_2
        const bool in_range = nrm >= 0x1p-60f && nrm <= 0x1p60f;
        const bool zero_row = all_zero(bits);
        if (!(in_range || zero_row)) w_sane = false;
        const float sc = in_range ? norm_scale(nrm) : 1.0f;
        // A row of zeros gives y = +0 for every pixel (bit 1), but its estimate 0 would never
        // be decided.  Such a row gets a weight on the first padded k, where every pixel
        // supplies the constant 1 (see BIAS_PAIR below): its estimate is 2^13, far above T.
        if (zero_row && ch < Co && KV == 16 * (BIAS_SLOT >> 3) + 8 * half + (BIAS_SLOT & 7))
            v[BIAS_SLOT] = 0x1p13f;
        row_unscale[m] = 1.0f / sc;
        rb = max(rb, __float_as_uint(nrm * sc));
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            uint32_t h4[4], l4[4];
#pragma unroll
            for (int d = 0; d < 4; ++d)
                split_pair(v[8 * t + 2 * d] * sc, v[8 * t + 2 * d + 1] * sc, h4[d], l4[d]);
            Wh[m][t] = make_uint4(h4[0], h4[1], h4[2], h4[3]);
            Wl[m][t] = make_uint4(l4[0], l4[1], l4[2], l4[3]);
        }
    }
    // wave maximum of the scaled row norms (unsigned order of the bit patterns of non-negative
    // floats is their numeric order) and wave-wide sanity of the rows
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) rb = max(rb, (uint32_t)__shfl_xor((int)rb, o));
    const float Wn = __uint_as_float(rb);
    w_sane = __builtin_amdgcn_ballot_w64(!w_sane) == 0;

    // ---- per-lane table of the NS gathered patch values: byte offset from the pixel and
    // which border makes the tap fall outside the image
    uint32_t off4[NS];
    uint32_t m_up = 0, m_dn = 0, m_lf = 0, m_rt = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = 16 * (s >> 3) + 8 * half + (s & 7);
        const int kk = k < KV ? k : 0;
        const int tap = kk / CI, ci = kk - tap * CI;
        const int ky = tap / 3, kx = tap - 3 * ky;
        off4[s] = k < KV ? (uint32_t)(((long)ci * H * W + (long)(ky - 1) * W + (kx - 1)) * 4) : OOB;
        if (k < KV) {
            m_up |= (ky == 0 ? 1u : 0u) << s;
            m_dn |= (ky == 2 ? 1u : 0u) << s;
            m_lf |= (kx == 0 ? 1u : 0u) << s;
            m_rt |= (kx == 2 ? 1u : 0u) << s;
        }
    }
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)img, 0, (int)img_bytes, 0x00020000);

    const int Cow = Co >> 5;
    const uint32_t psel = half ? 0x07060302u : 0x05040100u;
    const int widx = chunk * 2 + half;
    // geometry of a tile for this lane, and the gather of its patch values (0.0f outside the image)
    struct Geo { int y, n, x, xc; uint32_t pb; };
    auto geometry = [&](const TilePos &tp) {
        Geo g;
        g.y = tp.ty; g.n = tp.n;
        g.x = tp.tx * 32 + col;
        g.xc = min(g.x, W - 1);
        g.pb = (uint32_t)((((size_t)g.n * CI * H + g.y) * W + g.xc) * 4);
        return g;
    };
    auto gather = [&](const TilePos &tp, const Geo &g, float (&v)[NS]) {
        const bool interior = g.y > 0 && g.y < H - 1 && tp.tx > 0 && tp.tx * 32 + 32 < W;
        if (interior) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                v[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, g.pb + off4[s], 0, 0));
        } else {
            const uint32_t inv = (g.y == 0 ? m_up : 0u) | (g.y == H - 1 ? m_dn : 0u) |
                                 (g.xc == 0 ? m_lf : 0u) | (g.xc == W - 1 ? m_rt : 0u);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const uint32_t o = ((inv >> s) & 1u) ? OOB : g.pb + off4[s];
                v[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o, 0, 0));
            }
        }
    };

    // The operand planes of a tile: its patch values scaled to norm [2^12, 2^13) and split;
    // nx = scaled norm of the pixel's patch (0 for an all-zero patch, +inf when there is no
    // bound: non-finite or extreme values).  Built in pieces (see `tile`).
    struct Planes { uint4 h[KT], l[KT]; float nx, sc; };
    struct SplitState { float n2; uint32_t orb; float sc; };
    constexpr int NPIECE = 4 + NS / 2;
    auto split_piece = [&](int p, const float (&v)[NS], SplitState &st, Planes &P, uint32_t (&sh)[NS / 2],
                           uint32_t (&sl)[NS / 2]) {
        if (p == 0) {                       // squared norm of this lane's share, first half
            st.n2 = 0.0f;
#pragma unroll
            for (int s = 0; s < NS / 2; ++s) st.n2 = __builtin_fmaf(v[s], v[s], st.n2);
            asm volatile("" : "+v"(st.n2));
        } else if (p == 1) {                // ... second half
#pragma unroll
            for (int s = NS / 2; s < NS; ++s) st.n2 = __builtin_fmaf(v[s], v[s], st.n2);
            asm volatile("" : "+v"(st.n2));
        } else if (p == 2) {                // OR of the bit patterns: exact test for an all-zero patch
            st.orb = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) st.orb |= __float_as_uint(v[s]);
            asm volatile("" : "+v"(st.orb));
        } else if (p == 3) {                // both halves of the patch; the patch's scale
            const float nrm = __builtin_sqrtf(swap_add(st.n2));
            const bool zero = all_zero(st.orb);
            const bool in_range = nrm >= 0x1p-60f && nrm <= 0x1p60f;
            st.sc = in_range ? norm_scale(nrm) : 1.0f;
            P.nx = zero ? 0.0f : (in_range ? nrm * st.sc : __builtin_inff());
            P.sc = st.sc;
            asm volatile("" : "+v"(st.sc), "+v"(P.nx));
        } else {                            // one pair of values: scale, split
            const int q = p - 4;
            split_pair(v[2 * q] * st.sc, v[2 * q + 1] * st.sc, sh[q], sl[q]);
            asm volatile("" : "+v"(sh[q]), "+v"(sl[q]));
        }
    };
    // the constant 1.0 (fp16) at the padded term k = KV of every pixel: its slot reads 0.0f
    const uint32_t bias_or = half == BIAS_HALF ? (0x3c00u << (16 * (BIAS_SLOT & 1))) : 0u;
    auto finish_planes = [&](Planes &P, uint32_t (&sh)[NS / 2], const uint32_t (&sl)[NS / 2]) {
        sh[BIAS_SLOT / 2] |= bias_or;
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            P.h[t] = make_uint4(sh[4 * t], sh[4 * t + 1], sh[4 * t + 2], sh[4 * t + 3]);
            P.l[t] = make_uint4(sl[4 * t], sl[4 * t + 1], sl[4 * t + 2], sl[4 * t + 3]);
        }
    };

    // One tile: issue the loads of the tile after next, run the matrix instructions of the
    // current tile (operand planes B) with the scaling and split of the next tile's values
    // (vs -> Bn) cut into pieces, one after each matrix instruction - vector work is hidden only
    // between matrix instructions of the same wave - then decide and store.  Two sets of load
    // registers and two sets of operand planes alternate.
    TilePos ahead = tile_pos(slot, tstep.tiles_x, tstep.tiles_y);   // (tile in row, row, image)
    int tl_ahead = slot;                                           // tile index `ahead` stands for
    auto advance_ahead = [&]() {                                   // a wave's last tiles fetch themselves again
        if (tl_ahead + nslots < ntiles) { ahead.advance(tstep); tl_ahead += nslots; }
    };
    auto tile = [&](const Planes &B, Planes &Bn, float (&vs)[NS], float (&vl)[NS], const TilePos &pcur) {
        advance_ahead();
        gather(ahead, geometry(ahead), vl);
        const Geo gcur = geometry(pcur);

        // (the empty statements pin the loaded values to this iteration and "use" each piece's
        // results, so that the pieces stay between the matrix instructions as written)
#pragma unroll
        for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(vs[s]));
        v16f acc[2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[m][i] = 0.0f;
        SplitState st;
        uint32_t sh[NS / 2], sl[NS / 2];
        int piece = 0, issued = 0;
        auto mma = [&](const uint4 (&WP)[2][KT], const uint4 (&BP)[KT]) {
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_v8h(WP[m][t]), as_v8h(BP[t]), acc[m], 0, 0, 0);
                    ++issued;
                    __builtin_amdgcn_sched_barrier(0);
                    // one piece per matrix instruction, two while more pieces than instructions are left
                    if (piece < NPIECE) split_piece(piece++, vs, st, Bn, sh, sl);
                    if (piece < NPIECE && NPIECE - piece > 6 * KT - issued) split_piece(piece++, vs, st, Bn, sh, sl);
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        // small terms first; the two channel tiles alternate, so consecutive matrix
        // instructions never depend on each other
        mma(Wl, B.h);
        mma(Wh, B.l);
        mma(Wh, B.h);
#pragma unroll
        for (; piece < NPIECE; ++piece) split_piece(piece, vs, st, Bn, sh, sl);
        finish_planes(Bn, sh, sl);

        // ---- decision threshold of this pixel (scaled units; nx = +inf: no bound)
        const int y = gcur.y, n = gcur.n, x = gcur.x, xc = gcur.xc;
        const bool zero = B.nx == 0.0f;               // every patch value is +-0
        const float T = w_sane ? STEM_KAPPA * Wn * B.nx : __builtin_inff();
        float mn = __builtin_fminf(__builtin_fabsf(acc[0][0]), __builtin_fabsf(acc[0][1]));
#pragma unroll
        for (int i = 2; i < 16; ++i) mn = __builtin_fminf(mn, __builtin_fabsf(acc[0][i]));
        if (tile1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) mn = __builtin_fminf(mn, __builtin_fabsf(acc[1][i]));
        }
        // (non-finite estimates need no test of their own: they only arise from non-finite
        // or extreme inputs, which make T infinite)
        const bool flag = x < W && !zero && !(mn > T);

        // ---- sign bits (1 = negative) of the 2 x 16 channels of this lane
        uint32_t sg[2] = {0u, 0u};
#pragma unroll
        for (int i = 15; i >= 0; --i)
#pragma unroll
            for (int m = 0; m < 2; ++m)
                sg[m] = __builtin_amdgcn_alignbit(sg[m], __float_as_uint(acc[m][i]), 31);

        const size_t pix = ((size_t)n * H + y) * W + xc;
        if (WRITE_PRE) {
            // the estimates in the units of the inputs: undo the (exact) scales of pixel and rows
            // (the row scales live in other lanes: fetched with every lane active)
            const float ux = 1.0f / B.sc;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int cb = chunk * 64 + m * 32 + 16 * half;
                float o16[16];
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    o16[i] = acc[m][i] * ux * __shfl(row_unscale[m], tile_channel_to_row(16 * half + i));
                if (x < W && cb < Co) {
                    float4 *dst = reinterpret_cast<float4 *>(pre + pix * Co + cb);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        dst[q] = zero ? make_float4(0.0f, 0.0f, 0.0f, 0.0f)
                                      : make_float4(o16[4 * q], o16[4 * q + 1], o16[4 * q + 2], o16[4 * q + 3]);
                }
            }
        }

        // ---- sequential route for the undecided outputs (rare)
        if (__builtin_amdgcn_ballot_w64(flag) != 0) {
            if (WRITE_PRE) __builtin_amdgcn_s_waitcnt(0);   // the estimates are stored before the corrections
            if (flag) {
                // which outputs are undecided
                uint32_t fl[2];
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    fl[m] = 0;
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        fl[m] |= (!(__builtin_fabsf(acc[m][i]) > T) ? 1u : 0u) << i;
                    if (chunk * 64 + m * 32 + 16 * half >= Co) fl[m] = 0;
                }
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int cb = chunk * 64 + m * 32 + 16 * half;
                    while (fl[m]) {
                        const int i = __builtin_ctz(fl[m]);
                        fl[m] &= fl[m] - 1;
                        const float *wp = w + (size_t)(cb + i) * KV;
                        // the sum in its defined order, one kernel row (3 * CI terms) at a time;
                        // a tap outside the image is skipped, as in the definition
                        float s = 0.0f;
#pragma unroll
                        for (int ky = 0; ky < 3; ++ky) {
                            float pv[3 * CI], wv[3 * CI];
                            uint32_t okm = 0;
#pragma unroll
                            for (int e = 0; e < 3 * CI; ++e) {
                                const int kx = e / CI, ci = e - kx * CI;
                                const bool ok = !((ky == 0 && y == 0) || (ky == 2 && y == H - 1) ||
                                                  (kx == 0 && xc == 0) || (kx == 2 && xc == W - 1));
                                const uint32_t o = gcur.pb + (uint32_t)(((long)ci * H * W + (long)(ky - 1) * W + (kx - 1)) * 4);
                                pv[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, ok ? o : OOB, 0, 0));
                                wv[e] = wp[ky * 3 * CI + e];
                                okm |= (ok ? 1u : 0u) << e;
                            }
#pragma unroll
                            for (int e = 0; e < 3 * CI; ++e) {
                                const float f = __builtin_fmaf(wv[e], pv[e], s);
                                s = ((okm >> e) & 1u) ? f : s;
                            }
                        }
                        sg[m] = (sg[m] & ~(1u << i)) | ((s >= 0.0f ? 0u : 1u) << i);   // NaN -> bit 0
                        if (WRITE_PRE) pre[pix * Co + cb + i] = s;
                    }
                }
            }
        }
        if (zero) { sg[0] = 0u; sg[1] = 0u; }   // a chain of zero terms ends at +0.0f
        const uint32_t word = finish_word64(sg[0], sg[1], psel);
        if (x < W && widx < Cow) out[pix * Cow + widx] = word;
    };

    float va[NS], vb[NS];
    Planes B0, B1;
    TilePos p0 = ahead;
    gather(p0, geometry(p0), va);
    {
        SplitState st;
        uint32_t sh[NS / 2], sl[NS / 2];
#pragma unroll
        for (int p = 0; p < NPIECE; ++p) split_piece(p, va, st, B0, sh, sl);
        finish_planes(B0, sh, sl);
    }
    advance_ahead();
    TilePos p1 = ahead;
    gather(p1, geometry(p1), va);
    for (int tl = slot; tl < ntiles; tl += 2 * nslots) {
        tile(B0, B1, va, vb, p0);
        p0 = p1;
        p1 = ahead;
        if (tl + nslots >= ntiles) break;
        tile(B1, B0, vb, va, p0);
        p0 = p1;
        p1 = ahead;
    }
}

// ---------------------------------------------------------------------------------------
// Row-walking variant for three image channels.
//
// The kernel above gathers and splits all 27 values of every patch although a value belongs
// to nine patches.  Here a wave walks down a strip of 32 pixel columns; lane p owns halo pixel p, and
// a row is scaled and split ONCE, when it enters the window, and handed through wave-private LDS (four
// slots of one row) to the patches of the three rows it belongs to.  Sharing the split values means
// sharing the scale: instead of one power of two per patch the strip has one power of two s.  It is
// chosen to bring the largest magnitude of a window (3 rows x 34 pixels x 3 channels) into [2^11, 2^12)
// and kept while every row that enters stays below 2^15 (fp16 does not overflow) and one of three
// reaches 2^3, scaled; otherwise the wave chooses again and stages the window's older rows once more (a
// fetch of two rows, about 1 us; ordinary images do it a few times at most).  The error budget of the
// estimate changes in one place: the remainder of the split is bounded by 2^-22 |v| + 2^-25
// (the second term is the spacing of fp16 subnormals), and with a patch that is small against
// its window the absolute term no longer vanishes against the patch norm.  It is therefore part
// of the decision threshold:
//     T = kappa * max_o ||w_o|| * ||s x_patch||  +  2^-9
// (sum_k |w_k| 2^-25 <= sqrt(27) 2^13 2^-25 = 1.3e-3 < 2^-9 for rows scaled to a norm below
// 2^13, whatever s).  Outputs with |estimate| <= T take the sequential route as before, so the bits are
// those of the definition whatever the data; patches below about 2^-4, scaled (2^15 below the window's largest
// magnitude where the scale was chosen, 2^7 at the lower end to which it is kept), go down that route more often.  Windows with an infinity, or with a
// largest magnitude below 2^-111, get T = +inf.  The squared patch norm is the
// sum of three per-pixel sums of three rows exchanged through LDS; a NaN in it makes T NaN and the
// comparison fail, which is the sequential route again.
//
// K order of the matrix instruction (32 terms = 16 dwords of two fp16 values; lane (j, h) of a
// B operand supplies dwords 8t + 4h + d of block t): a slot holds two dwords per halo pixel p and plane -
// P[p] = channels (0, 1), Z[p] = channel 2 of pixels (p, p + 1) - and pixel j reads, for window rows 0 .. 2,
//     h = 0:  P0[j] P0[j+1] Z0[j] Z0[j+1]  |  P0[j+2] P1[j+2]    P1[j] P1[j+1]
//     h = 1:  P2[j] P2[j+1] Z2[j] Z2[j+1]  |  P2[j+2] (1.0, 0)   Z1[j] Z1[j+1]
// (the first value of a Z[j+1] meets weight 0).  The constant gives an all-zero weight row, and the rows beyond Co,
// an estimate that is decided wherever the kept scale stands (SR_BIAS).  The weights are loaded in the same order, and no value moves between
// registers: every dword is read where the matrix instruction wants it.
//
// What bounds it: about 107 vector and 12 matrix instructions a tile, which overlap by a tenth.  Staging a row
// once instead of three times took 175 -> 107 vector instructions.  1024x2048 36.7 -> 32.6 us back to back, 32x640x959 303 -> 265, 8x1024x1024 to 128 channels
// 252 -> 222, 512x512 10.1 -> 9.6 (three waves per SIMD).  Measured and not kept: four waves per SIMD (31.9 us alone, but the layers
// behind it get slower, see stem_segment_rows); the decision of row y - 1 between the matrix instructions of row y (a
// second set of accumulators, two waves per SIMD): 38.4 us.  The undecided outputs (6 % of the tiles have one)
// are listed and summed 64 at a time, all taps of a sum fetched at once from one base offset, and a block's
// waves share the preparation of the weights, behind the fetches of the first image rows.  A tile with many
// undecided outputs (non-finite or tiny windows, a weight row out of range, dense ties) sums them in the lanes
// that hold them, a pixel's patch fetched once for all of them: with every output undecided 512x1024 x 64 takes
// 123 us, with 200 NaN pixels 46, ordinary data 15 (a patch fetched again for every output, a kernel row at a
// time: 560 and 392).
constexpr int SR_HW = 34;                    // halo pixels of a strip
constexpr int SR_ARR = 36;                   // dwords per LDS array (34 used)
constexpr int SR_Z = SR_ARR;                 // from P of a plane to its Z
constexpr int SR_LO = 2 * SR_ARR;            // from the plane of the leading terms to that of the remainders
constexpr int SR_SLOT = 4 * SR_ARR;          // P and Z of both planes: one image row
constexpr int SR_CONST = SR_ARR - 1;         // spare dword of P: the constant entry
constexpr int SR_N = 4 * SR_SLOT;            // per halo pixel: squared norm of its three rows
constexpr int SR_Q = SR_N + SR_ARR;          // undecided outputs that wait for their sequential sums
constexpr int SR_QCAP = 192;
constexpr int SR_WAVE = SR_Q + SR_QCAP;      // dwords per wave
constexpr float SR_FLOOR = 0x1p-9f;
// Estimate of a row of zeros.  It has to exceed the largest threshold of a finite window: rows of a norm below
// 2^13 (1.002: the margin in KW) against 27 values below 2^15
constexpr float SR_BIAS = 0x1p15f;
static_assert(SR_BIAS > STEM_KAPPA * 1.003f * 0x1p13f * 5.1962f * 0x1p15f + SR_FLOOR, "a row of zeros is decided everywhere");

// index into the 27 weights of an output channel for half h, dword dh = 4t + d, fp16 value e;
// -1: no term (weight 0), -2: the constant term
__host__ __device__ constexpr int sr_term(int h, int dh, int e)
{
    const int ky = h == 0 ? 0 : 2;                                   // window row of dwords 0 .. 4
    if (dh < 2 || dh == 4) return (ky * 3 + (dh < 2 ? dh : 2)) * 3 + e;
    if (dh == 2) return (ky * 3 + e) * 3 + 2;
    if (dh == 3) return e ? (ky * 3 + 2) * 3 + 2 : -1;
    if (h == 0) return (1 * 3 + (dh == 5 ? 2 : dh - 6)) * 3 + e;
    if (dh == 5) return e == 0 ? -2 : -1;
    if (dh == 6) return (1 * 3 + e) * 3 + 2;
    return e ? (1 * 3 + 2) * 3 + 2 : -1;
}

// maximum over the wave of a value that is the same non-negative number in no particular lane
// order (0 is the identity): shifts inside rows of 16 lanes, then lane 15 of a row into the
// next row, lane 31 into the upper half; lane 63 holds the result
__device__ __forceinline__ uint32_t wave_umax(uint32_t x)
{
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true));   // row_shr:1
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true));   // row_shr:2
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true));   // row_shr:4
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true));   // row_shr:8
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));  // row_bcast:15
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

__global__ __launch_bounds__(256, 2) void stem_rows_kernel(
    const float *__restrict__ img, uint32_t img_bytes, int H, int W, const float *__restrict__ w, int Co,
    int nchunks, int strips, int nseg, int seg_rows, int units, uint32_t *__restrict__ out)
{
    constexpr int KV = 27;
    __shared__ uint32_t lds[4][SR_WAVE];
    __shared__ uint4 wts[2][2][2][64];         // [hi, lo][tile][block of K][lane]
    __shared__ uint32_t wnorm[2], winsane[2];  // per tile: largest scaled norm; a norm out of range

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk = blockIdx.x % nchunks;    // 64 output channels of the block
    const int gw = blockIdx.x / nchunks * 4 + wave;
    int q = min(gw, units - 1);                // (surplus waves: addresses of the last unit)
    const int sx = q % strips; q /= strips;        // strip of 32 pixel columns
    const int sg = q % nseg;                       // segment of seg_rows image rows
    const int n = q / nseg;
    const int col = lane & 31, half = lane >> 5;
    const int y0 = sg * seg_rows;
    const int rows = min(H, y0 + seg_rows) - y0;
    const int x0 = sx * 32;

    // ---- addresses.  Staging: lane p < 34 owns halo pixel p (image column x0 - 1 + p); the
    // other lanes repeat pixel 33.  Zero padding: a column or row outside the image gets an
    // offset beyond the buffer and reads 0.0f.
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)img, 0, (int)img_bytes, 0x00020000);
    const int p = min(lane, SR_HW - 1);
    const int xs = x0 - 1 + p;
    const uint32_t xoff = (xs >= 0 && xs < W) ? (uint32_t)xs * 4u : OOB;
    uint32_t *const ldsw = lds[wave];
    // image row y0 - 1 + k of the strip lives in slot k % 4
    uint32_t *const wr = ldsw + p;
    // row y - 1 (lower half) and row y + 1 (upper half), two slots further: [first slot even / 2]
    const uint32_t *const qa[2] = {ldsw + col + (half ? 2 * SR_SLOT : 0), ldsw + col + (half ? 0 : 2 * SR_SLOT)};
    const uint32_t *const qb = ldsw + col + (half ? SR_Z : 0);               // row y: P | Z
    const uint32_t *const qc = ldsw + (half ? SR_CONST : col + 2);           // row y: P[j + 2] | the constant
    if (lane < 4) {
        ldsw[lane * SR_SLOT + SR_CONST] = 0x3c00u;       // (1.0, 0) in the leading plane, 0 in the other
        ldsw[lane * SR_SLOT + SR_CONST + SR_LO] = 0u;
    }

    const int Cow = Co >> 5;
    const uint32_t psel = half ? 0x07060302u : 0x05040100u;
    const int widx = chunk * 2 + half;
    const int xo = x0 + col;                   // output pixel column of this lane
    // packed output of image n as a buffer: lane offset inside a row, row offset per tile
    const uint32_t out_row_bytes = (uint32_t)W * Cow * 4u;
    const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(out + (size_t)n * H * W * Cow), 0, (int)(H * out_row_bytes), 0x00020000);
    // (validity goes into the row offset alone: two out-of-range marks would add up to 0)
    const uint32_t out_voff = (uint32_t)(xo * Cow + widx) * 4u;

    struct Planes { uint4 h[2], l[2]; float ns[3]; bool ok; };   // operands of a tile, norms of its columns

    // one image row of the strip: three floats per lane
    auto fetch = [&](int yy, float (&v)[3]) {
        const bool rin = yy >= 0 && yy < H;
        const int yc = min(max(yy, 0), H - 1);
        const uint32_t vo = rin ? xoff : OOB;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            v[c] = __uint_as_float(
                __builtin_amdgcn_raw_buffer_load_b32(rsrc, vo, (int)((((size_t)n * 3 + c) * H + yc) * W * 4), 0));
    };
    // rows y0 - 1 .. y0 + 1 for the first tile, rows y0 + 2 and y0 + 3: under way while the weights are prepared
    float a[3][3], ld0[3], ld1[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) fetch(y0 - 1 + r, a[r]);
    fetch(y0 + 2, ld0);
    fetch(y0 + 3, ld1);

    // ---- weights: rows scaled to a norm in [2^12, 2^13), split once, in the K order above.  Wave w
    // prepares tile w & 1, block w >> 1 of K (the norm needs the whole row) and the block shares them:
    // a quarter of the 32 splits each, which is what a short segment otherwise spends its time on.
    {
        const int m = wave & 1, t = wave >> 1;
        const int ch = chunk * 64 + m * 32 + tile_row_to_channel(col);
        float v[16];
        float part = 0.0f;
        uint32_t bits = 0;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int k0 = sr_term(0, s >> 1, s & 1), k1 = sr_term(1, s >> 1, s & 1);
            const int k = half ? k1 : k0;
            const bool ok = ch < Co && k >= 0;
            const float wv = w[ok ? (size_t)ch * KV + k : 0];   // unconditional load
            v[s] = ok ? wv : 0.0f;
            part = __builtin_fmaf(v[s], v[s], part);
            bits |= __float_as_uint(v[s]);
        }
        const float nrm = __builtin_sqrtf(swap_add(part));
        const bool zero_row = all_zero(bits);
        const bool in_range = nrm >= 0x1p-60f && nrm <= 0x1p60f;
        const float sc = in_range ? norm_scale(nrm) : 1.0f;
        if (zero_row && half == 1) v[10] = SR_BIAS;              // the constant term (dword 5)
        uint32_t h4[4], l4[4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
            split_pair((t ? v[8 + 2 * d] : v[2 * d]) * sc, (t ? v[9 + 2 * d] : v[2 * d + 1]) * sc, h4[d], l4[d]);
        wts[0][m][t][lane] = make_uint4(h4[0], h4[1], h4[2], h4[3]);
        wts[1][m][t][lane] = make_uint4(l4[0], l4[1], l4[2], l4[3]);
        const uint32_t rb = wave_umax(__float_as_uint(nrm * sc));
        const bool insane = __builtin_amdgcn_ballot_w64(!(in_range || zero_row)) != 0;
        if (t == 0 && lane == 0) {
            wnorm[m] = rb;
            winsane[m] = insane ? 1u : 0u;
        }
    }
    __syncthreads();
    if (gw >= units) return;                   // whole wave leaves; nothing is shared from here on
    uint4 Wh[2][2], Wl[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            Wh[m][t] = wts[0][m][t][lane];
            Wl[m][t] = wts[1][m][t][lane];
        }
    // (margin: the patch norm is good to 2^-10)
    const float KW = STEM_KAPPA * 1.002f * __uint_as_float(max(wnorm[0], wnorm[1]));
    const bool w_sane = (winsane[0] | winsane[1]) == 0;

    // ---- the strip's power of two: s brings the largest magnitude of a window into [2^11, 2^12).  It stays
    // while every row that enters is below `hi` (2^15 scaled) and one of three reaches `lo` (2^3 scaled)
    float sc_s = 1.0f, sc_hi = 0.0f, sc_lo = 0.0f;
    bool sc_ok = false;
    auto pick_scale = [&](uint32_t rm) {       // rm: largest magnitude, as bits
        const uint32_t e = rm >> 23;
        const bool in_range = e >= 16u && e <= 254u;
        sc_ok = in_range || rm == 0u;          // (all zero: any scale)
        sc_s = in_range ? __uint_as_float((265u - e) << 23) : 1.0f;
        sc_hi = in_range ? __uint_as_float(min(e + 4u, 255u) << 23) : 0x1p-110f;
        sc_lo = in_range ? __uint_as_float((e - 8u) << 23) : 0.0f;
    };
    auto row_bits = [](const float (&v)[3]) {
        return max(max(__float_as_uint(v[0]) & 0x7fffffffu, __float_as_uint(v[1]) & 0x7fffffffu),
                   __float_as_uint(v[2]) & 0x7fffffffu);
    };
    // trailing rows of a window that do not reach sc_lo under the scale just chosen for it (one of the three does)
    auto rows_below = [&](const float (&v1)[3], const float (&v2)[3]) {
        const uint32_t lo = __float_as_uint(sc_lo);
        return __builtin_amdgcn_ballot_w64(row_bits(v2) >= lo) != 0 ? 0 : __builtin_amdgcn_ballot_w64(row_bits(v1) >= lo) != 0 ? 1 : 2;
    };
    auto split2 = [](v2f f, uint32_t &hi, uint32_t &lo) {
        hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2h));
        // f - hi (exact: the difference has at most 24 bits) with the fp16 operand converted by
        // the instruction itself: -1.0 * hi.lo + f[0], -1.0 * hi.hi + f[1]
        v2f r;
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r[0]) : "v"(hi), "v"(f[0]));
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r[1]) : "v"(hi), "v"(f[1]));
        lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2h));
    };
    // One row: scaled, split, written to its slot; returns the squared norm of this pixel's values (channels 0
    // and 1 from the leading fp16 terms: 2^-10 relative, covered by the margin in KW; what rounds to zero there
    // is below 2^-24 and covered by the constant part of the threshold).  Zero only if the three values are.
    struct Stage { float x[4], m; uint32_t ph, pl, zh, zl; };
    auto scale_row = [&](const float (&v)[3], float m, Stage &st) {
        st.m = m;
#pragma unroll
        for (int c = 0; c < 3; ++c) st.x[c] = v[c] * sc_s;
        // channel 2 of the next pixel (lanes beyond the halo repeat its last pixel: nobody reads what they write)
        st.x[3] = __uint_as_float(
            (uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(st.x[2]), 0x130, 0xf, 0xf, true));
        asm volatile("" : "+v"(st.x[0]), "+v"(st.x[1]), "+v"(st.x[2]), "+v"(st.x[3]));
    };
    auto write_row = [&](const Stage &st, uint32_t *dst) {
        dst[0] = st.ph;
        dst[SR_Z] = st.zh;
        dst[SR_LO] = st.pl;
        dst[SR_LO + SR_Z] = st.zl;
        const v2h h = __builtin_bit_cast(v2h, st.ph);
        const float n2 = __builtin_fmaf(st.x[2], st.x[2], __builtin_amdgcn_fdot2(h, h, 0.0f, false));
        return __uint_as_float(max(__float_as_uint(n2), min(__float_as_uint(st.m), 0x0d800000u)));   // 2^-100
    };
    float n_prev = 0.0f, n_pair = 0.0f;        // norm of the row that entered last, and of the last two together
    auto stage_row = [&](const float (&v)[3], uint32_t *dst) {
        Stage st;
        scale_row(v, __uint_as_float(row_bits(v)), st);
        split2((v2f){st.x[0], st.x[1]}, st.ph, st.pl);
        split2((v2f){st.x[2], st.x[3]}, st.zh, st.zl);
        return write_row(st, dst);
    };

    // Staging of the row that enters (it completes the window of the next tile, whose first row is in slot K)
    // and the next tile's operands, in pieces
    constexpr int STAGE_PIECES = 7;
    auto stage_piece = [&](auto kk, int slot, const float (&v)[3], float m, Stage &st, Planes &Bn) {
        constexpr int K = decltype(kk)::value;
        if (slot == 0) {
            scale_row(v, m, st);
        } else if (slot == 1) {
            split2((v2f){st.x[0], st.x[1]}, st.ph, st.pl);
            asm volatile("" : "+v"(st.ph), "+v"(st.pl));
        } else if (slot == 2) {
            split2((v2f){st.x[2], st.x[3]}, st.zh, st.zl);
            asm volatile("" : "+v"(st.zh), "+v"(st.zl));
        } else if (slot == 3) {
            const float n = write_row(st, wr + (K + 2) % 4 * SR_SLOT);
            ldsw[SR_N + p] = __float_as_uint(n_pair + n);
            n_pair = n_prev + n;
            n_prev = n;
            __builtin_amdgcn_wave_barrier();
        } else if (slot < 6) {
            // LDS instructions of a wave execute in order: these reads see the writes above
            const int pl = (slot - 4) * SR_LO;
            const uint32_t *const a = qa[K / 2] + K % 2 * SR_SLOT + pl;
            const uint32_t *const b = qb + (K + 1) % 4 * SR_SLOT + pl, *const c = qc + (K + 1) % 4 * SR_SLOT + pl;
            uint4(&out)[2] = slot == 4 ? Bn.h : Bn.l;
            out[0] = make_uint4(a[0], a[1], a[SR_Z], a[SR_Z + 1]);
            out[1] = make_uint4(a[2], c[0], b[0], b[1]);
        } else {
            // the three columns of this lane's patch; the threshold is formed where it is used
#pragma unroll
            for (int d = 0; d < 3; ++d) Bn.ns[d] = __uint_as_float(ldsw[SR_N + col + d]);
            Bn.ok = sc_ok;
            __builtin_amdgcn_wave_barrier();   // the next row is written after these reads
        }
    };

    // the sum of one output in its defined order (ky, kx, ci), term u = (ky * 3 + kx) * 3 + ci; a tap outside the
    // image is skipped
    struct Pixel { uint32_t off; bool up, dn, lf, rt; };   // offset in channel 0; has a neighbour on that side
    auto pixel = [&](int y, int x) {
        return Pixel{(uint32_t)((((size_t)n * 3 * H + y) * W + x) * 4), y > 0, y < H - 1, x > 0, x < W - 1};
    };
    auto inside = [](int u, const Pixel &px) {
        const int ky = u / 9, kx = u % 9 / 3;
        return (ky == 1 || (ky == 0 ? px.up : px.dn)) && (kx == 1 || (kx == 0 ? px.lf : px.rt));
    };
    auto patch = [&](const Pixel &px, float (&pv)[KV]) {
#pragma unroll
        for (int u = 0; u < KV; ++u) {
            const uint32_t o = px.off + (uint32_t)(((u % 3 * H + u / 9 - 1) * W + u % 9 / 3 - 1) * 4);
            pv[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, inside(u, px) ? o : OOB, 0, 0));
        }
    };
    auto chain = [&](const Pixel &px, const float (&pv)[KV], int ch) {
        const float *const wp = w + (size_t)ch * KV;
        float wv[KV], sum = 0.0f;
#pragma unroll
        for (int u = 0; u < KV; ++u) wv[u] = wp[u];   // in one batch
#pragma unroll
        for (int u = 0; u < KV; ++u) {
            const float f = __builtin_fmaf(wv[u], pv[u], sum);
            sum = inside(u, px) ? f : sum;
        }
        return sum;
    };
    int qn = 0;   // entries of the list of undecided outputs
    // ---- decision and store of a finished row
    struct Done { float T; bool zero; int i; };
    struct Epi { float mn; uint32_t sg; };     // bit b of sg: sign of register b % 16 of tile b / 16
    constexpr int EPI_PIECES = 7;
    auto epi_piece = [&](int k, const v16f (&acc)[2], const Done &dn, Epi &ep) {
        if (k == 0) {
            float mn = __builtin_fminf(__builtin_fabsf(acc[0][0]), __builtin_fabsf(acc[0][1]));
#pragma unroll
            for (int e = 2; e < 16; ++e) mn = __builtin_fminf(mn, __builtin_fabsf(acc[0][e]));
            ep.mn = mn;
            ep.sg = 0u;
            asm volatile("" : "+v"(ep.mn));
        } else if (k == 1) {
            float mn = ep.mn;
#pragma unroll
            for (int e = 0; e < 16; ++e) mn = __builtin_fminf(mn, __builtin_fabsf(acc[1][e]));
            ep.mn = mn;
            asm volatile("" : "+v"(ep.mn));
        } else if (k < 6) {
            // sign bits (1 = negative) of the 2 x 16 channels of this lane, eight per piece
#pragma unroll
            for (int e = 31 - 8 * (k - 2); e > 23 - 8 * (k - 2); --e)
                ep.sg = __builtin_amdgcn_alignbit(ep.sg, __float_as_uint(acc[e >> 4][e & 15]), 31);
            asm volatile("" : "+v"(ep.sg));
        } else {
            const int y = y0 + dn.i;
            const float T = dn.T;
            const bool live = xo < W && dn.i >= 0 && dn.i < rows;
            const bool flag = live && !dn.zero && !(ep.mn > T);
            // ---- sequential route for the undecided outputs (rare): a few of them are put on the wave's
            // list and summed later, one per lane, instead of in the lane that found them with 63 idle
            // (their bits are provisional until then); a tile with many (unusual data) sums in place
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(flag) != 0, 0)) {
                uint32_t fl[2] = {0, 0};
                if (flag)
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            fl[m] |= (!(__builtin_fabsf(acc[m][e]) > T) ? 1u : 0u) << e;
                        if (chunk * 64 + m * 32 + 16 * half >= Co) fl[m] = 0;
                    }
                uint32_t todo = fl[0] | fl[1] << 16;
                if (__builtin_popcountll(__builtin_amdgcn_ballot_w64(todo != 0)) <= 16 &&
                    __builtin_amdgcn_ballot_w64(__builtin_popcount(todo) > 4) == 0) {
                    uint64_t who;
                    while ((who = __builtin_amdgcn_ballot_w64(todo != 0)) != 0) {
                        if (todo) {
                            const int b = __builtin_ctz(todo);
                            todo &= todo - 1;
                            const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0));
                            // channel of the chunk: tile b / 16, half, register b % 16
                            ldsw[SR_Q + qn + at] =
                                (uint32_t)dn.i << 11 | (uint32_t)((b >> 4) * 32 + 16 * half + (b & 15)) << 5 | (uint32_t)col;
                        }
                        qn += __builtin_popcountll(who);
                    }
                } else if (flag) {
                    // the patch is fetched once for all of the pixel's outputs
                    const Pixel px = pixel(y, xo);
                    float pv[KV];
                    patch(px, pv);
                    uint32_t neg = 0;
                    for (uint32_t left = todo; left; left &= left - 1) {
                        const int b = __builtin_ctz(left);
                        const float sum = chain(px, pv, chunk * 64 + (b >> 4) * 32 + 16 * half + (b & 15));
                        neg |= (sum >= 0.0f ? 0u : 1u) << b;   // NaN -> bit 0
                    }
                    ep.sg = (ep.sg & ~todo) | neg;
                }
            }
            const uint32_t mine = dn.zero ? ~0u : ~ep.sg;   // a chain of zero terms ends at +0.0f
            const auto sw = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);
            const uint32_t word = __builtin_amdgcn_perm(sw[1], sw[0], psel);
            const uint32_t roff = live && widx < Cow ? (uint32_t)y * out_row_bytes : OOB;
            __builtin_amdgcn_raw_buffer_store_b32(word, orsrc, out_voff + roff, 0, 0);
        }
    };

    // ---- one tile: matrix instructions of row y on planes B, between them the staging of row y + 2 (fetched
    // two tiles ago) for the tile below; then decision and store.  K: slot of row y, the first of the next window.
    // (Running the decision of row y - 1 between the matrix instructions as well, with a second set of
    // accumulators, measured slower, 38.4 us at 1024x2048: the kernel is bound by the vector instruction count.)
    int low = 0;                               // rows in a row that did not reach sc_lo
    auto tile = [&](auto kk, const int i, const Planes &B, Planes &Bn, float (&ld)[3]) {
        constexpr int K = decltype(kk)::value;
        const int y = y0 + i;
        const float m = __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(ld[0]), __builtin_fabsf(ld[1])),
                                        __builtin_fabsf(ld[2]));
        low = __builtin_amdgcn_ballot_w64(m >= sc_lo) != 0 ? 0 : low + 1;
        if (__builtin_expect(!sc_ok || low >= 3 || __builtin_amdgcn_ballot_w64(!(m < sc_hi)) != 0, 0)) {
            // another scale: the window's other two rows once more (unless this row has none either)
            const uint32_t own = wave_umax(row_bits(ld)) >> 23;
            if (sc_ok || own == 0u || (own >= 16u && own <= 254u)) {
                float r0[3], r1[3];
                fetch(y, r0);
                fetch(y + 1, r1);
                pick_scale(wave_umax(max(max(row_bits(r0), row_bits(r1)), row_bits(ld))));
                n_pair = stage_row(r0, wr + K * SR_SLOT);
                n_prev = stage_row(r1, wr + (K + 1) % 4 * SR_SLOT);
                n_pair += n_prev;
                low = rows_below(r1, ld);
            }
        }

        v16f acc[2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][e] = 0.0f;
        Stage st;
        Epi ep;
        Done dn;
        int slot = 0;
        auto mma = [&](const uint4 (&WP)[2][2], const uint4 (&BP)[2]) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int mm = 0; mm < 2; ++mm) {
                    acc[mm] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_v8h(WP[mm][t]), as_v8h(BP[t]), acc[mm], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (slot < STAGE_PIECES) stage_piece(kk, slot, ld, m, st, Bn);
                    if (slot == 0) fetch(y + 4, ld);
                    ++slot;
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        // (a wave in its matrix instructions goes ahead of waves in their vector instructions: 33.7 -> 32.8 us at
        // 1024x2048, 267.6 -> 262.1 at 32x640x959; launch bounds of two waves per SIMD leave three room, 159 registers)
        __builtin_amdgcn_s_setprio(1);
        mma(Wl, B.h);      // small terms first
        mma(Wh, B.l);
        mma(Wh, B.h);
        __builtin_amdgcn_s_setprio(0);
        static_assert(STAGE_PIECES <= 12, "one piece per matrix instruction");

        const float n2 = B.ns[0] + B.ns[1] + B.ns[2];
        dn.zero = __float_as_uint(n2) == 0u;                          // every patch value is +-0
        // (the hardware square root is good to 1 ulp; KW carries the margin)
        dn.T = (B.ok && w_sane) ? __builtin_fmaf(KW, __builtin_amdgcn_sqrtf(n2), SR_FLOOR) : __builtin_inff();
        dn.i = i;
#pragma unroll
        for (int k = 0; k < EPI_PIECES; ++k) epi_piece(k, acc, dn, ep);
    };

    // ---- prologue: rows y0 - 1 .. y0 + 1 staged for the first tile
    Planes B0, B1;
    {
        pick_scale(wave_umax(max(max(row_bits(a[0]), row_bits(a[1])), row_bits(a[2]))));
        n_pair = stage_row(a[0], wr);
        n_prev = stage_row(a[1], wr + SR_SLOT);
        n_pair += n_prev;
        low = rows_below(a[1], a[2]);
        Stage st;
        const float m = __uint_as_float(row_bits(a[2]));
#pragma unroll
        for (int k = 0; k < STAGE_PIECES; ++k) stage_piece(std::integral_constant<int, 0>{}, k, a[2], m, st, B0);
    }
    // the listed outputs, one per lane
    auto flush = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the words with the provisional bits are out
        for (int b = 0; b < qn; b += 64)
            if (b + lane < qn) {
                const uint32_t en = ldsw[SR_Q + b + lane];
                const int y = y0 + (int)(en >> 11), x = x0 + (int)(en & 31u), ch = chunk * 64 + (int)(en >> 5 & 63u);
                const Pixel px = pixel(y, x);
                float pv[KV];
                patch(px, pv);
                const float sum = chain(px, pv, ch);
                uint32_t *const word = out + (((size_t)n * H + y) * W + x) * Cow + (ch >> 5);
                if (sum >= 0.0f) atomicOr(word, 1u << (ch & 31));
                else atomicAnd(word, ~(1u << (ch & 31)));   // NaN -> bit 0
            }
        qn = 0;
    };
    // four rows per trip: operand planes and fetch registers alternate, the slots rotate.  A row lists at most
    // 64 outputs.
#pragma unroll 1
    for (int i = 0; i < rows; i += 4) {
        if (__builtin_expect(qn > SR_QCAP - 128, 0)) flush();
        tile(std::integral_constant<int, 1>{}, i, B0, B1, ld0);
        if (i + 1 >= rows) break;
        tile(std::integral_constant<int, 2>{}, i + 1, B1, B0, ld1);
        if (i + 2 >= rows) break;
        if (__builtin_expect(qn > SR_QCAP - 128, 0)) flush();
        tile(std::integral_constant<int, 3>{}, i + 2, B0, B1, ld0);
        if (i + 3 >= rows) break;
        tile(std::integral_constant<int, 0>{}, i + 3, B1, B0, ld1);
    }
    if (qn) flush();
}

// Rows of a segment: as many segments as it takes to give every wave slot of the chip one unit, with three waves
// per SIMD, but with two where these segments would have 8 to 31 rows.  The layer alone takes the same time with
// either (1024x2048 33.1 us with three, 33.7 with two, 8x480x640 38.4 and 39.5), but a network runs at the clock that
// its power leaves it, and on frames that are not in the caches three waves cost every layer behind this one
// 1 to 2 % of its clock (four 3 %).  Networks of 64 channels on changing frames, us with three -> with two:
// 720x1280 369.8 -> 359.5, 1024x2048 604.4 -> 591.1, 4x480x640 466.8 -> 454.1, 8x480x640 (26 rows) 805.8 -> 796.1,
// 3x720x1280 (30 rows) 838.0 -> 829.1.  Where segments are longer three are better: 2x1024x2048 (44 rows) 1039.9 ->
// 1045.8, 16x480x640 (54) 1395.6 -> 1404.3, and the layer alone, 32x640x959 268 -> 282, 8x1024x1024 to 128 channels
// 225 -> 235.  Three with 32 channels too, whose networks leave power: 720x1280 161.1 -> 162.4, the layer alone 16.1 ->
// 17.0, and where segments are shorter: their passes are short of waves, not of power (480x640 195.0 and 194.9), and the
// layer alone loses when its few rows are rounded up (2x186x334 to 128 channels, 4 -> 6 rows, 9.8 -> 10.8).
static int stem_segment_rows(int H, int Co, long base)
{
    auto rows = [&](long waves_per_simd) {
        const int r = ceil_div(H, (int)std::max(1L, waves_per_simd * 4 * 256 / base));
        return std::max(2, r + (r & 1));
    };
    return rows(3) >= 8 && rows(3) < 32 && Co > 32 ? rows(2) : rows(3);
}

static int launch_stem_rows(const float *img, uint32_t bytes, int N, int H, int W, const float *w, int Co,
                            uint32_t *out_bits, hipStream_t s)
{
    const int nchunks = ceil_div(Co, 64);
    const int strips = ceil_div(W, 32);
    const long base = (long)N * strips * nchunks;
    const int seg_rows = stem_segment_rows(H, Co, base);
    const int nseg = ceil_div(H, seg_rows);
    const long units = (long)N * strips * nseg;   // of every chunk
    if (units > 0x7fffffffL || (units + 3) / 4 * nchunks > 0x7fffffffL) return fail(MBU_ERR_SHAPE, "stem: too many tiles for one launch");
    MBU_LAUNCH(stem_rows_kernel, dim3((unsigned)((units + 3) / 4 * nchunks)), dim3(256), 0, s, img, bytes, H, W, w, Co,
               nchunks, strips, nseg, seg_rows, (int)units, out_bits);
    return check_launch("stem_rows");
}


int launch_stem_mfma(const float *img, int N, int Ci, int H, int W, const float *w, int Co,
                     uint32_t *out_bits, float *out_pre, hipStream_t s)
{
    const double bytes = (double)N * Ci * H * W * 4.0;
    if (bytes >= 2147483648.0) return fail(MBU_ERR_SHAPE, "stem: image larger than 2 GiB");
    // (the row-walking kernel addresses the packed output of one image with 31-bit offsets)
    if (Ci == 3 && !out_pre && t_cfg.stem_path != MBU_STEM_MFMA_GATHER && (double)(H + 1) * (W + 32) * (Co / 32) * 4.0 < 2147483648.0)
        return launch_stem_rows(img, (uint32_t)bytes, N, H, W, w, Co, out_bits, s);
    const int tiles_x = ceil_div(W, 32);
    const long ntiles = (long)N * H * tiles_x;
    if (ntiles > 0x7fffffffL) return fail(MBU_ERR_SHAPE, "stem: too many tiles for one launch");
    const int nchunks = ceil_div(Co, 64);
    // two waves per SIMD over the whole chip (what the register budget allows), so all waves
    // are resident at once; every wave keeps one 64-channel chunk
    const int max_waves = 2 * 4 * 256;
    if (nchunks > max_waves) return fail(MBU_ERR_SHAPE, "stem: too many output channels");
    const int nslots = (int)min(ntiles, (long)(max_waves / nchunks));
    const int waves = nslots * nchunks;
    const TileStep tstep = tile_step(nslots, tiles_x, H);
    const dim3 grid(ceil_div(waves, 4)), block(256);
#define MBU_STEM_LAUNCH(CI, PRE)                                                                    \
    MBU_LAUNCH((stem_mfma_kernel<CI, PRE>), grid, block, 0, s, img, (uint32_t)bytes, N, H, W, w, Co, \
               nchunks, nslots, (int)ntiles, tstep, out_bits, out_pre)
    if (Ci == 3) {
        if (out_pre) MBU_STEM_LAUNCH(3, true); else MBU_STEM_LAUNCH(3, false);
    } else if (Ci == 1) {
        if (out_pre) MBU_STEM_LAUNCH(1, true); else MBU_STEM_LAUNCH(1, false);
    } else {
        return fail(MBU_ERR_SHAPE, "stem supports 1 or 3 image channels, got %d", Ci);
    }
#undef MBU_STEM_LAUNCH
    return check_launch("stem_mfma");
}

}  // namespace mbu
