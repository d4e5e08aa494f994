// Layer-by-layer ResNet path: BOTH residual blocks of a section in one launch, the residual stream in registers.
//
// resnet_strip.h's kernel holds one convolution's output in accumulators and lets x make a trip to memory per block: on
// maps cut into strips that is two launches, each reading the stream twice and writing it (fp32 between them).  Here a
// workgroup has a compute unit to itself - eight wavefronts of 256 registers - so that x stays in fp32 registers next
// to the accumulators from the first block's input to the second block's output.  HBM sees the pooled map (bf16) once on
// the way in, with the halo rows that neighbouring strips share, and the section's output once on the way out.
//
// The map is resnet_strip.h's: planar bf16, rows of W + 1 cells with one shared zero cell as both borders, walked flat,
// rewritten in place by every convolution.  All four convolutions walk the SAME pixel tiles - the rows the first one
// covers, three more than the strip on every inner side - so that a pixel is the same lane's throughout and its x can
// stay where it is; the outer rows hold nothing valid any more after a convolution or two and are never read for a pixel
// that is stored.  Workgroups are persistent, and the next strip's pixels arrive beside the map (asynchronous loads, as
// they lie in memory) from the last convolution's end on.
//
// Measured in one run, 1024 images, us, two launches of strips with x in memory -> this one: 32 channels on 36 x 48 (two strips of 18
// rows) 233 -> 172; 16 channels on 54 x 72 233 -> 146; 64 channels on 18 x 24 161 -> 131, on 9 x 12 64 -> 40; 128 on 9 x 12 170 ->
// 131 (in the agents' steps 156, 134, 118, 35 and 119).  In the order found (32 channels on 36 x 48): everything the epilogues and the x phase know about a pixel
// worked out once per strip shape, not per phase (a wavefront's two vector instructions per pixel and phase are its time:
// 184 -> 171 us); a lane's feature tiles one run of eight channels, so that a cell is one 16-byte access;
// fragments of all of a wavefront's tiles requested ahead (ring of 9 instead of 3); the next convolution's first weights
// requested before the epilogue; loops written out, not indexed by the block (a pointer picked at run time makes its
// loads flat ones, which count as LDS traffic too: 171 -> 165).
// What bounds it (32 channels on 36 x 48): by counters the matrix cores are busy 46 % of the time (56 % at 64 channels, 68 % at 128);
// the rest is mostly the epilogues between the convolutions, vector instructions that no MFMA covers because all eight
// wavefronts pass them together, and the fragments' first trip behind each barrier.
// Random data also lowers the clock: the same launches on zeros take 7 - 17 % less.
#pragma once
#include <algorithm>

#include "resnet_strip.h"

namespace seedinf {

constexpr int RP_THREADS = 512;
constexpr size_t RP_LDS_MAX = 160 * 1024;                   // one workgroup per compute unit
constexpr int RP_MAX_STACK = 4;                             // images a workgroup stacks

template <int C>
struct PairCfg {
    using S = StripCfg<C>;
    // pixel tiles a wavefront holds x and accumulators for (at 16 channels in steps of two): 144 - 160 registers
    static constexpr int TPW = C == 16 ? 18 : (C == 128 ? 10 : 9);
    static constexpr int MAX_TILES = TPW * S::NPG;
    static constexpr size_t map_bytes(int rows, int W) { return S::lds_bytes(rows + 2, W); }
    // the incoming map: whole kilobytes
    static constexpr size_t raw_bytes(int pixels) { return ((size_t)pixels * C * 2 + 1023) / 1024 * 1024; }
    // (a tile's lanes past the end of the map read up to 15 cells behind it: the incoming map)
    static constexpr size_t lds_bytes(int rows, int pixels, int W) { return map_bytes(rows, W) + raw_bytes(pixels); }
    static constexpr bool fits(int rows, int pixels, int W)
    {
        return S::tiles(rows, W) <= MAX_TILES && lds_bytes(rows, pixels, W) <= RP_LDS_MAX;
    }
    // 16-byte pieces of the incoming map's pixels are rotated within the pixel so that one piece of 16 consecutive pixels
    // falls on 256 distinct bank bytes: where piece q of pixel px is
    __device__ static __forceinline__ int piece(int px, int q) { return px * S::NCG + ((q + px * S::NCG / 16) & (S::NCG - 1)); }
};

struct PairArgs {
    const __bf16* x_in;                // [B, H, W, C]: the pooled map
    const bf16x8* wp[4];               // conv_a, conv_b of the first and of the second block
    const float* bias[4];
    __bf16* y;                         // the second block's output
    int y_relu, ldy;                   // rectify y; ldy > 0: y is the feature matrix [B, ldy], (h, w, c) order
    int B, H, W, TH, strips;           // strips of TH rows per image; strips == 1 with `stack` images per workgroup
    int stack, items, rows;            // items: strips or stacks of the batch; rows: the most a convolution covers
};

struct PairPlan {
    int TH = 0, strips = 0;            // TH == 0: no strip fits
    long cells = 0;                    // map cells the four convolutions walk over all strips of an image
    static int conv_rows(int th, int ns) { return ns == 1 ? th : (ns == 2 ? th + 3 : th + 6); }
    // pixels of the incoming map: the rows a convolution covers and one more on every inner side
    static int in_rows(int th, int ns) { return ns == 1 ? th : (ns == 2 ? th + 4 : th + 8); }
    // The fewest strips that fit: the halo rows are what a strip costs.
    template <int C>
    bool choose(int H, int W)
    {
        for (int ny = 1; ny <= H; ++ny) {
            const int th = (H + ny - 1) / ny, ns = (H + th - 1) / th;
            const int r = std::min(conv_rows(th, ns), H), n = std::min(in_rows(th, ns), H);
            if (!PairCfg<C>::fits(r, n * W, W)) continue;
            TH = th; strips = ns;
            cells = 4L * ns * PairCfg<C>::S::tiles(r, W) * 16;
            return true;
        }
        return false;
    }
    int rows(int H, int stack) const { return stack > 1 ? stack * (H + 1) - 1 : std::min(conv_rows(TH, strips), H); }
    int pixels(int H, int W, int stack) const { return stack > 1 ? stack * H * W : std::min(in_rows(TH, strips), H) * W; }
    // Images of one strip that a workgroup stacks: the fewest tiles in whole rounds over the compute units, a round's own
    // cost (barriers, the trips behind them) counted as a third of the tiles a wavefront can hold.  Measured with every
    // stack forced, 15 networks at 200 to 2500 images: this one within 0.2 % of the best on average (4.6 % at most), stacks
    // made while every compute unit keeps a workgroup within 5.5 % (23 %): those leave 257 to 511 images two rounds of one image
    // (16 channels on 9 x 12, 300 images: step 24.9 -> 20.9 us, 1000: 30.7 -> 26.0; 64 on 13 x 13, 640: 83 -> 72).
    template <int C>
    int stack(int B, int H, int W, int n_cu) const
    {
        using K = PairCfg<C>;
        if (strips != 1) return 1;
        int images = 1;
        long best = 0;
        for (int s = 1; s <= RP_MAX_STACK && (s == 1 || K::fits(s * (H + 1) - 1, s * H * W, W)); ++s) {
            const int workgroups = (B + s - 1) / s, tiles = (K::S::tiles(s * (H + 1) - 1, W) + K::S::NPG - 1) / K::S::NPG;
            const long cost = (long)((workgroups + n_cu - 1) / n_cu) * (K::TPW / 3 + tiles);
            if (s == 1 || cost < best) { best = cost; images = s; }
        }
        return images;
    }
};

// by_tiles for this kernel's counts: at 16 channels even ones (an odd count computes its last pixel tile once more)
template <int C, class F>
__device__ __forceinline__ void by_pair_tiles(int nt, F phase)
{
    auto go = [&](auto ntc) {
        if constexpr (decltype(ntc)::value <= PairCfg<C>::TPW) phase(ntc);
    };
    constexpr int K = C == 16 ? 2 : 1;
    switch ((min(nt, PairCfg<C>::TPW) + K - 1) / K) {
    case 0: go(std::integral_constant<int, 0>{}); break;
    case 1: go(std::integral_constant<int, 1 * K>{}); break;
    case 2: go(std::integral_constant<int, 2 * K>{}); break;
    case 3: go(std::integral_constant<int, 3 * K>{}); break;
    case 4: go(std::integral_constant<int, 4 * K>{}); break;
    case 5: go(std::integral_constant<int, 5 * K>{}); break;
    case 6: go(std::integral_constant<int, 6 * K>{}); break;
    case 7: go(std::integral_constant<int, 7 * K>{}); break;
    case 8: go(std::integral_constant<int, 8 * K>{}); break;
    case 9: go(std::integral_constant<int, 9 * K>{}); break;
    case 10: go(std::integral_constant<int, 10 * K>{}); break;
    }
}

template <int C>
__global__ __launch_bounds__(RP_THREADS, 2) void resblock_pair_kernel(PairArgs p)
{
    using K = PairCfg<C>;
    using S = StripCfg<C>;
    constexpr int FTW = S::FTW, NCG = S::NCG, CPL = 4 * FTW;
    typedef __bf16 lane_bf16 __attribute__((ext_vector_type(CPL)));         // a lane's channels of a pixel
    extern __shared__ __attribute__((aligned(16))) char rp_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int P = p.W + 1, Hp = p.H + 1;
    const bool stacked = p.stack > 1;
    const int PL = S::plane(p.rows + 2, p.W);
    const size_t img = (size_t)p.H * p.W * C;
    char* const map = rp_lds;
    char* const raw = rp_lds + NCG * PL * 16;
    const uint32_t raw_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)raw;

    // consecutive workgroups land on the eight XCDs in turn: each XCD walks one run of consecutive strips, whose shared
    // halo rows then meet in its L2
    const int xcd = blockIdx.x & 7, wgs = ((int)gridDim.x - xcd + 7) >> 3;
    const int per = p.items >> 3, rem = p.items & 7;
    const int lo = xcd * per + min(xcd, rem), hi = lo + per + (xcd < rem ? 1 : 0);

    // an item's strip: image b (and nimg - 1 more), rows y0 .. ye - 1; map row 0 is image row m0, the first convolution covers
    // `ra` rows from map row 1 on; the incoming map starts at image row t0 and has npx pixels
    struct Item { int b, y0, ye, m0, ra, nimg, t0, npx; };
    auto item_at = [&](int it) {
        Item t;
        t.b = stacked ? it * p.stack : it / p.strips;
        t.y0 = stacked ? 0 : (it % p.strips) * p.TH;
        t.ye = min(t.y0 + p.TH, p.H);
        t.nimg = min(p.stack, p.B - t.b);
        t.m0 = max(t.y0 - 4, -1);
        t.ra = stacked ? t.nimg * Hp - 1 : min(t.ye + 3, p.H) - (t.m0 + 1);
        t.t0 = max(t.m0, 0);
        t.npx = stacked ? t.nimg * p.H * p.W : (min(t.ye + 4, p.H) - t.t0) * p.W;
        return t;
    };
    // asynchronous loads of an item's pixels, a contiguous kilobyte an instruction (past the end: the last pixel again)
    auto issue = [&](const Item& t) {
        const int ln = fresh_lane(lane);
        const __bf16* src = p.x_in + t.b * img + (size_t)t.t0 * p.W * C;
        for (int k = wave; k * (64 / NCG) < t.npx; k += 8) {
            const int px = k * (64 / NCG) + ln / NCG, q = (ln % NCG - px * NCG / 16) & (NCG - 1);
            g2lds16(src + (size_t)min(px, t.npx - 1) * C + q * 8, raw_at + k * 1024);
        }
    };

    const int first = lo + (blockIdx.x >> 3);
    if (first >= hi) return;
    issue(item_at(first));
    // the border cells, and the rows between stacked images, are never written again
    for (int k = tid; k < NCG * PL; k += RP_THREADS) *(bf16x8*)(map + k * 16) = bf16x8{};
    const int fg = wave % S::NFG, pg = wave / S::NFG;
    const int npa = p.rows * P - 1;                          // pixels the convolutions walk
    // the row on either side of the walked ones: R = ReLU(x), zero outside the image (always there in a stack)
    auto edge_rows = [&](const Item& t) {
        if (stacked) return;
        for (int k = tid; k < 2 * p.W * NCG; k += RP_THREADS) {
            const int q = k % NCG, c2 = k / NCG, lower = c2 >= p.W, c = c2 - (lower ? p.W : 0);
            const int r = lower ? t.ra + 1 : 0, y = t.m0 + r;
            bf16x8 v = {};
            if (y >= 0 && y < p.H) {
                v = *(const bf16x8*)(raw + K::piece((y - t.t0) * p.W + c, q) * 16);
                const bf16x4 l = relu_bf16x4(__builtin_shufflevector(v, v, 0, 1, 2, 3));
                const bf16x4 h = relu_bf16x4(__builtin_shufflevector(v, v, 4, 5, 6, 7));
                v = __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7);
            }
            *(bf16x8*)(map + (q * PL + r * P + 1 + c) * 16) = v;
        }
    };
    // the lane's channels in the map: plane and byte in the cell
    auto cell_of = [&](int ln) {
        const int g = ln >> 4, q = P + 1 + pg * 16 + (ln & 15);
        return map + (FTW == 2 ? ((fg * 4 + g) * PL + q) * 16 : ((g >> 1) * PL + q) * 16 + (g & 1) * 8);
    };
    by_pair_tiles<C>(((npa + 15) / 16 - pg + S::NPG - 1) / S::NPG, [&](auto ntc) {
        constexpr int NT = decltype(ntc)::value, NA = NT > 0 ? NT : 1, RING = NA > 9 ? NA / 2 : (NA == 9 && C >= 64 ? 3 : NA);
        // per tile, the lanes whose pixel is one of an image, and those whose pixel is the strip's; the lane's piece of
        // the incoming map (two to a register)
        uint64_t inside[NA], mine[NA];
        uint32_t at[(NA + 1) / 2];
        int y0 = -1, nimg = 0;                               // the strip these belong to
        const bf16x8* wl[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) wl[k] = p.wp[k] + fg * FTW * S::KCH * 64;
        StripWeights<C, C >= 64 ? 3 : 2> w;
        for (int it = first;;) {
            const Item t = item_at(it);
            const int next = it + wgs;
            if (NT > 0 && (t.y0 != y0 || t.nimg != nimg)) {
                y0 = t.y0; nimg = t.nimg;
                const int ln = fresh_lane(lane), g = ln >> 4, q = FTW == 2 ? fg * 4 + g : g >> 1;
                TileWalk tw(pg * 16 + (ln & 15), S::NPG * 16, P);
#pragma unroll
                for (int i = 0; i < NT; ++i, tw.next()) {
                    int y = t.m0 + 1 + tw.r, im = 0;         // row and image of the stack
                    if (stacked) {
#pragma unroll
                        for (int k = 1; k < RP_MAX_STACK; ++k)
                            if (y >= Hp) { y -= Hp; ++im; }
                    }
                    // (a stack's separating rows have y = H)
                    const bool in = tw.r < t.ra && tw.c < p.W && y < p.H;
                    inside[i] = __ballot(in);
                    mine[i] = __ballot(in && y >= t.y0 && y < t.ye);
                    const uint32_t pc = in ? K::piece((im * p.H + y - t.t0) * p.W + tw.c, q) : 0;
                    if (i % 2 == 0) at[i / 2] = pc;
                    else at[i / 2] |= pc << 16;
                }
            }
            auto piece_at = [&](int i) { return (at[i / 2] >> (16 * (i % 2))) & 0xffffu; };
            stage_wait();
            __syncthreads();                                 // the pixels have landed, and everybody has left the previous map
            edge_rows(t);
            if constexpr (NT == 0) {
                // the other wavefronts' barriers: behind x, and two per convolution but the last
                for (int k = 0; k < 7; ++k) __syncthreads();
                if (next < hi) issue(item_at(next));
            } else {
                floatx4 x[NT][FTW];
                // a pixel's rectified values into the map (border cells keep their zeros)
                auto put = [&](char* cell, int i, const floatx4 (&v)[FTW]) {
                    bf16x4 r[FTW];
#pragma unroll
                    for (int j = 0; j < FTW; ++j) r[j] = relu_bf16x4(to_bf16x4(v[j]));
                    if (__builtin_amdgcn_inverse_ballot_w64(inside[i])) {
                        if constexpr (FTW == 2) *(bf16x8*)cell = __builtin_shufflevector(r[0], r[1], 0, 1, 2, 3, 4, 5, 6, 7);
                        else *(bf16x4*)cell = r[0];
                    }
                };
                // ---- x, and R ----
                {
                    const int ln = fresh_lane(lane);
                    const char* from = raw + (FTW == 2 ? 0 : (ln >> 4 & 1) * 8);
                    lane_bf16 v[NT];
#pragma unroll
                    for (int i = 0; i < NT; ++i) v[i] = *(const lane_bf16*)(from + piece_at(i) * 16);
                    w.start(wl[0], ln);
                    char* cell = cell_of(ln);
#pragma unroll
                    for (int i = 0; i < NT; ++i, cell += S::NPG * 256) {
                        bf16x4 r[FTW];
#pragma unroll
                        for (int j = 0; j < FTW; ++j) {
                            const bf16x4 u = j == 0 ? __builtin_shufflevector(v[i], v[i], 0, 1, 2, 3) : __builtin_shufflevector(v[i], v[i], CPL - 4, CPL - 3, CPL - 2, CPL - 1);
                            x[i][j] = to_floatx4(u);
                            r[j] = relu_bf16x4(u);
                        }
                        if (__builtin_amdgcn_inverse_ballot_w64(inside[i])) {
                            if constexpr (FTW == 2) *(bf16x8*)cell = __builtin_shufflevector(r[0], r[1], 0, 1, 2, 3, 4, 5, 6, 7);
                            else *(bf16x4*)cell = r[0];
                        }
                    }
                }
                __syncthreads();
                auto convolve = [&](int conv, floatx4 (&acc)[NT][FTW], floatx4 (&bv)[FTW], auto tail) {
                    const int g = fresh_lane(lane) >> 4;
#pragma unroll
                    for (int j = 0; j < FTW; ++j) bv[j] = *(const floatx4*)(p.bias[conv] + fg * FTW * 16 + g * CPL + j * 4);
                    strip_conv<C, NT, RING>(map, PL, P, pg, npa - 1, wl[conv], lane, w, acc, tail);
                };
                floatx4 acc[NT][FTW], bv[FTW];
                // (every convolution requests the next one's first weights before its epilogue)
                auto rewrite = [&](int conv, auto value) {
                    convolve(conv, acc, bv, [] {});
                    w.start(wl[conv + 1], fresh_lane(lane));
                    char* cell = cell_of(fresh_lane(lane));
                    __syncthreads();                         // everybody has read the map
#pragma unroll
                    for (int i = 0; i < NT; ++i, cell += S::NPG * 256) {
#pragma unroll
                        for (int j = 0; j < FTW; ++j) value(i, j);
                        put(cell, i, acc[i]);
                    }
                    __syncthreads();
                };
                auto conv_a = [&](int i, int j) { acc[i][j] += bv[j]; };                                 // U = ReLU(conv_a(R) + bias)
                auto conv_b = [&](int i, int j) { acc[i][j] = x[i][j] = acc[i][j] + bv[j] + x[i][j]; };  // x' = x + conv_b(U) + bias, R = ReLU(x')
                rewrite(0, conv_a);
                rewrite(1, conv_b);
                rewrite(2, conv_a);
                // (the incoming map is free since x was read)
                convolve(3, acc, bv, [&] { if (next < hi) issue(item_at(next)); });
                const int ln = fresh_lane(lane);
                __bf16* const out = p.y + (p.ldy > 0 ? (size_t)t.b * p.ldy : t.b * img) + (size_t)t.t0 * p.W * C + fg * FTW * 16 + (ln >> 4) * CPL;
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    bf16x4 r[FTW];
#pragma unroll
                    for (int j = 0; j < FTW; ++j) {
                        r[j] = to_bf16x4(acc[i][j] + bv[j] + x[i][j]);
                        if (p.y_relu) r[j] = relu_bf16x4(r[j]);
                    }
                    const int px = piece_at(i) / NCG;
                    int to = px * C;
                    if (p.ldy > 0 && stacked) to += px / (p.H * p.W) * (p.ldy - (int)img);       // (rows of the feature matrix may be padded)
                    if (__builtin_amdgcn_inverse_ballot_w64(mine[i])) {
                        if constexpr (FTW == 2) *(bf16x8*)(out + to) = __builtin_shufflevector(r[0], r[1], 0, 1, 2, 3, 4, 5, 6, 7);
                        else *(bf16x4*)(out + to) = r[0];
                    }
                }
            }
            if (next >= hi) return;
            it = next;
        }
    });
}

}  // namespace seedinf
