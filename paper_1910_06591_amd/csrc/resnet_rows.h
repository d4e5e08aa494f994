// First layer of the layer-by-layer ResNet path with its 3x3 / stride-2 max-pool, uint8 frame -> x as bf16, pooled down
// the rows in registers.
//
// A workgroup takes full-width strips of pooled rows.  A wavefront walks down a column strip of 16 pixels: the lane
// that holds a pixel holds the pixels below it too, so the vertical maximum of three convolution rows is one instruction
// per value on the accumulators, one row shared with the next pooled row, and bias, scale, rounding and the trip to LDS
// are paid on pooled rows only.  (The maximum commutes with all of those, so the bits are first_pool_kernel's, which pools
// rounded values from a convolution tile in LDS: of numbers below 2.6e36, the range of the packed maximum in both kernels.
// Sums that are infinite or NaN, from weights of that size, are carried by neither.)  The horizontal maximum takes three reads per pooled pixel instead
// of nine.  The weights stay in registers; workgroups are persistent, and the next strip's rows are on their way in
// registers while this one's are convolved.
//
// K layout and packed weights as in first_pool_kernel: frames of up to 4 planes in cells of 4 channels, chunk kc = kernel rows
// 2 kc and 2 kc + 1, two adjacent columns per lane group; 16 planes in two planes of 8 channels, k = tap * 16 + plane.
//
// Measured in one run, 1024 frames, us, against first_pool_kernel: 72 x 96 x 3 -> 32 channels 118 -> 72, -> 64 195 -> 143, -> 16
// 64 -> 40; 16 planes -> 16 channels on 108 x 144 212 -> 185, on 90 x 120 156 -> 121 (in the agents' steps 65, 135, -, 172 and
// 114; the rows ahead are worth 6 to 20 % of them).  By counters (72 x 96 x 3 -> 32; 108 x 144 x 16) the
// wavefronts wait 40 / 58 % of the time, mostly for each other at the two barriers of a strip: with 16 planes a strip is
// four pooled rows, four or five units of work to a wavefront.
// (The same kernel on the 16-channel bf16 input of a later section is no faster than strip_pool_kernel, 88 -> 87.)
#pragma once
#include <cfloat>

#include "resnet_strip.h"

namespace seedinf {

constexpr int FR_THREADS = 512;
constexpr size_t FR_LDS_MAX = 80 * 1024;                    // two workgroups per compute unit

struct FirstRowsArgs {
    const uint8_t* in;                 // frames [B, H, W, CIN]
    const bf16x8* wp;                  // [COUT / 16][chunks][64 lanes][8]
    const float* bias;
    float scale;                       // of the sums
    __bf16* x;                         // [B, PH, PW, COUT]
    int B, H, W, PH, PW, pad_h, pad_w, PTH, strips, groups;
};

template <int CIN, int COUT>
struct FirstRowsCfg {
    static constexpr bool CELL4 = CIN <= 4;
    static_assert(CELL4 || CIN == 16, "planes with a kernel");
    static_assert(COUT == 16 || COUT == 32 || COUT == 64, "output channels");
    static constexpr int KCH = CELL4 ? 2 : 5;
    static constexpr int FTW = COUT == 16 ? 1 : 2, NFG = COUT / 16 / FTW, NPW = 8 / NFG, NCG = COUT / 8;
    static constexpr int CELL = CELL4 ? 8 : 16, PLANES = CELL4 ? 1 : 2;
    // cells of an input plane: 2 PTH + 3 rows of W + 1, whose cell 0 is zero: the border of its own row and of the one
    // above; and the cells that the last row's windows reach into
    __host__ __device__ static constexpr int plane(int PTH, int W) { return ((2 * PTH + 3) * (W + 1) + 4 + 15) / 16 * 16; }
    __host__ __device__ static constexpr int in_bytes(int PTH, int W) { return PLANES * plane(PTH, W) * CELL; }
    // pooled rows before the horizontal maximum: planes of 8 channels, a row's even and odd columns apart, so that neither
    // 16 columns written nor 16 pooled pixels read fall on a bank twice; planes 256 / NCG bytes apart modulo 256, so that
    // the lanes that read all channels of a pixel do not either
    __host__ __device__ static constexpr int half(int W) { const int b = (W + 1) / 2 * 16; return (b + 127) / 256 * 256 + 128; }
    __host__ __device__ static constexpr int out_plane(int PTH, int W) { return PTH * 2 * half(W) + 256 / NCG; }
    static constexpr size_t lds_bytes(int PTH, int W) { return (size_t)in_bytes(PTH, W) + NCG * out_plane(PTH, W); }
    // input of a strip on its way in registers: items of four pixels (cells of 4 channels) or one, PRE to a thread
    static constexpr int PRE = CELL4 ? 2 : 4, DW = CELL4 ? CIN : 4;
    __host__ __device__ static constexpr int items(int rows, int W) { return rows * (CELL4 ? W / 4 : W); }
    // rows of pooled pixels per strip: the fewest convolution rows in all
    static bool choose(int PH, int W, int& PTH, int& strips)
    {
        long best = -1;
        for (int ns = 1; ns <= PH; ++ns) {
            const int th = (PH + ns - 1) / ns, n = (PH + th - 1) / th;
            if (lds_bytes(th, W) > FR_LDS_MAX || items(2 * th + 3, W) > PRE * FR_THREADS) continue;
            const long cost = (long)n * (2 * th + 4);
            if (best < 0 || cost < best) { best = cost; PTH = th; strips = n; }
        }
        return best >= 0 && (!CELL4 || W % 4 == 0);
    }
};

template <int CIN, int COUT>
__global__ __launch_bounds__(FR_THREADS, 4) void first_rows_kernel(FirstRowsArgs p)
{
    using K = FirstRowsCfg<CIN, COUT>;
    constexpr int KCH = K::KCH, FTW = K::FTW, NCG = K::NCG, CELL = K::CELL, PRE = K::PRE, DW = K::DW;
    extern __shared__ __attribute__((aligned(16))) char fr_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int P = p.W + 1, PL = K::plane(p.PTH, p.W), HS = K::half(p.W), OP = K::out_plane(p.PTH, p.W);
    char* const in = fr_lds;
    char* const out = fr_lds + K::in_bytes(p.PTH, p.W);

    // each XCD walks one run of consecutive strips (see resblock_pair_kernel)
    const int xcd = blockIdx.x & 7, wgs = ((int)gridDim.x - xcd + 7) >> 3;
    const int per = p.groups >> 3, rem = p.groups & 7;
    const int lo = xcd * per + min(xcd, rem), hi = lo + per + (xcd < rem ? 1 : 0);
    int it = lo + (blockIdx.x >> 3);
    if (it >= hi) return;

    // ---- a strip's input rows: requested one strip ahead, then written as bf16 (whole numbers of a frame exactly), zero
    // outside the frame ----
    const int WI = K::CELL4 ? p.W >> 2 : p.W;
    uint32_t d[PRE][DW];
    auto request = [&](int strip) {
        const int b = strip / p.strips, ph0 = (strip % p.strips) * p.PTH, rows = min(p.PTH, p.PH - ph0);
        const int items = (2 * rows + 3) * WI, yt = 2 * ph0 - p.pad_h - 1;
        const uint32_t* const frame = (const uint32_t*)p.in + (size_t)b * p.H * WI * DW;
        RowWalk rw(tid, FR_THREADS, WI);
#pragma unroll
        for (int u = 0; u < PRE; ++u, rw.next()) {
            // unconditional, from a clamped place in the frame: a select on what was loaded would wait for it here
            const int y = min(max(yt + rw.r, 0), p.H - 1);
            if (u * FR_THREADS < items) {                    // uniform
                const uint32_t* s = frame + (size_t)(y * WI + rw.c) * DW;
                if constexpr (DW % 4 == 0) {
#pragma unroll
                    for (int k = 0; k < DW; k += 4) *(uint4*)&d[u][k] = *(const uint4*)(s + k);
                } else {
#pragma unroll
                    for (int k = 0; k < DW; ++k) d[u][k] = s[k];
                }
            }
        }
    };
    auto write = [&](int strip) {
        const int ph0 = (strip % p.strips) * p.PTH, rows = min(p.PTH, p.PH - ph0);
        const int items = (2 * rows + 3) * WI, yt = 2 * ph0 - p.pad_h - 1;
        RowWalk rw(tid, FR_THREADS, WI);
#pragma unroll
        for (int u = 0; u < PRE; ++u, rw.next()) {
            if (tid + u * FR_THREADS >= items) continue;
            const int y = yt + rw.r;
            const bool inside = y >= 0 && y < p.H;
            if constexpr (K::CELL4) {
                char* cell = in + (rw.r * P + 1 + rw.c * 4) * 8;
#pragma unroll
                for (int px = 0; px < 4; ++px) {
                    floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < CIN; ++k) v[k] = (float)((d[u][(px * CIN + k) / 4] >> (8 * ((px * CIN + k) % 4))) & 0xffu);
                    const uint2 o = __builtin_bit_cast(uint2, to_bf16x4(v));
                    *(uint2*)(cell + px * 8) = inside ? o : uint2{0u, 0u};
                }
            } else {
                char* cell = in + (rw.r * P + 1 + rw.c) * 16;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint4 o = __builtin_bit_cast(uint4, u8x8_to_bf16x8(d[u][2 * h % DW], d[u][(2 * h + 1) % DW]));
                    *(uint4*)(cell + h * PL * 16) = inside ? o : uint4{0u, 0u, 0u, 0u};
                }
            }
        }
    };
    request(it);
    // the border cells and what lies behind the last row stay zero
    for (int k = tid; k < K::in_bytes(p.PTH, p.W) / 16; k += FR_THREADS) *(uint4*)(in + k * 16) = uint4{0u, 0u, 0u, 0u};

    const int fg = wave % K::NFG, pw = wave / K::NFG;
    // weights: with two feature tiles, eight consecutive channels per lane group (see StripWeights)
    bf16x8 a[KCH][FTW];
    {
        const int first = FTW == 2 ? ((n & 8) >> 3) * KCH * 64 + (lane & 48) + (n & 4) * 2 + (n & 3) : lane;
#pragma unroll
        for (int kc = 0; kc < KCH; ++kc)
#pragma unroll
            for (int j = 0; j < FTW; ++j) a[kc][j] = p.wp[fg * FTW * KCH * 64 + j * 4 + kc * 64 + first];
    }
    floatx4 bv[FTW];
#pragma unroll
    for (int j = 0; j < FTW; ++j) bv[j] = *(const floatx4*)(p.bias + fg * FTW * 16 + g * 4 * FTW + j * 4);
    int off[KCH];                                            // byte offset of a chunk's taps from the pixel's window
#pragma unroll
    for (int kc = 0; kc < KCH; ++kc) {
        if constexpr (K::CELL4) {
            off[kc] = ((kc == 0 ? (g >> 1) : 2) * P + 2 * (g & 1)) * 8;      // (chunk 1 of lane groups 2 and 3: zero weights)
        } else {
            const int tap = min(2 * kc + (g >> 1), 8);       // (the tenth tap has zero weights)
            off[kc] = ((g & 1) * PL + (tap / 3) * P + tap % 3) * 16;
        }
    }
    auto fragment = [&](const char* s) {
        if constexpr (K::CELL4) {                            // 8-byte aligned
            const bf16x4 l = *(const bf16x4*)s, h = *(const bf16x4*)(s + 8);
            return __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            return *(const bf16x8*)s;
        }
    };
    __syncthreads();
    write(it);
    for (;;) {
        const int next = it + wgs;
        const int b = it / p.strips, ph0 = (it % p.strips) * p.PTH, rows = min(p.PTH, p.PH - ph0);     // pooled rows
        __syncthreads();                                     // the rows are in, and everybody has left the previous strip's maxima
        if (next < hi) request(next);

        // ---- convolution rows, and their maxima over three rows ----
        const int units = ((p.W + 15) >> 4) * rows, u0 = pw * units / K::NPW, u1 = (pw + 1) * units / K::NPW;
        int cs = u0 / rows, py = u0 - cs * rows;             // column strip, pooled row
        bool fresh = true;
        floatx4 carry[FTW];
        const char* s = nullptr;
        char* o = nullptr;
        for (int u = u0; u < u1; ++u) {
            const int y = 2 * (ph0 + py) - p.pad_h;          // the frame's row of the window's first (uniform)
            if (fresh) {
                const int col = min(cs * 16 + n, p.W - 1);
                s = in + (2 * py * P + col) * CELL;
                o = out + py * 2 * HS + (col & 1) * HS + (col >> 1) * 16 + (FTW == 2 ? (fg * 4 + g) * OP : (g >> 1) * OP + (g & 1) * 8);
                // the first row: part of the pooled row unless it lies outside the frame
#pragma unroll
                for (int j = 0; j < FTW; ++j) carry[j] = y >= 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : floatx4{-FLT_MAX, -FLT_MAX, -FLT_MAX, -FLT_MAX};
                if (y >= 0) {
#pragma unroll
                    for (int kc = 0; kc < KCH; ++kc) {
                        const bf16x8 f = fragment(s + off[kc]);
#pragma unroll
                        for (int j = 0; j < FTW; ++j) carry[j] = mfma16(a[kc][j], f, carry[j]);
                    }
                }
                s += P * CELL;
            }
            floatx4 acc[2][FTW];
            bf16x8 f[2][KCH];
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int kc = 0; kc < KCH; ++kc) f[r][kc] = fragment(s + r * P * CELL + off[kc]);
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int j = 0; j < FTW; ++j) acc[r][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < KCH; ++kc)
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int j = 0; j < FTW; ++j) acc[r][j] = mfma16(a[kc][j], f[r][kc], acc[r][j]);
            bf16x4 v[FTW];
#pragma unroll
            for (int j = 0; j < FTW; ++j) {
                floatx4 m;
                if (y + 2 < p.H) {                           // uniform: the third row lies in the frame
#pragma unroll
                    for (int i = 0; i < 4; ++i) m[i] = fmaxf(fmaxf(carry[j][i], acc[0][j][i]), acc[1][j][i]);
                } else {
                    m = max4(carry[j], acc[0][j]);
                }
                carry[j] = acc[1][j];
                v[j] = to_bf16x4(m * p.scale + bv[j]);
            }
            if (cs * 16 + n < p.W) {
                if constexpr (FTW == 2) *(bf16x8*)o = __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7);
                else *(bf16x4*)o = v[0];
            }
            s += 2 * P * CELL;
            o += 2 * HS;
            fresh = ++py == rows;
            if (fresh) { py = 0; ++cs; }
        }
        __syncthreads();

        // ---- the next strip's rows, and maxima over three columns (those outside the frame clamped onto it) ----
        if (next < hi) write(next);
        const int npool = rows * p.PW;
        __bf16* const x = p.x + ((size_t)b * p.PH + ph0) * p.PW * COUT + (tid % NCG) * 8;
        RowWalk rw(tid / NCG, FR_THREADS / NCG, p.PW);
        const char* const pl = out + (tid % NCG) * OP;
        for (int px = tid / NCG; px < npool; px += FR_THREADS / NCG, rw.next()) {
            const char* const row = pl + rw.r * 2 * HS;
            auto at = [&](int c) {
                const int cc = min(max(c, 0), p.W - 1);
                return *(const uint4*)(row + (cc & 1) * HS + (cc >> 1) * 16);
            };
            const int c0 = 2 * rw.c - p.pad_w;
            *(uint4*)(x + (size_t)px * COUT) = bf16x8_max(bf16x8_max(at(c0), at(c0 + 1)), at(c0 + 2));
        }
        if (next >= hi) return;
        it = next;
    }
}

}  // namespace seedinf
