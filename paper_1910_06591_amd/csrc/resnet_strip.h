// Layer-by-layer ResNet path, maps whose full-width strips fit LDS and are the faster cut (strips_preferred in
// bf16_path.h): conv0 + pooling of a section, and its residual blocks, each in one launch over ONE LDS map that every
// convolution rewrites in place.  (Both blocks in one launch where their halo allows it: resnet_pair.h.)
//
// A workgroup takes TH rows of an image (all W columns).  The map is planar
// bf16 [C/8][cells][8 channels]; a row is W + 1 cells, cell 0 of which is zero: it is the left border of its own row
// and the right border of the row above (SAME padding without a second border column).  The output pixels of a
// convolution are walked flat over the map, border cells included (computed, and kept zero): a tile is 16
// consecutive cells, so its fragments are 256 distinct bank bytes - the full LDS rate, where 16 row-major pixels
// of a narrower region wrap rows and read at about 57 % - and tile i of a wavefront sits at a constant distance
// from tile 0: one address register for all of them, immediates for the rest.  (The staging writes are not free of
// conflicts: the lanes of a pixel hold its channel groups, whose planes lie whole 256 bytes apart.)
//
// In place: a wavefront keeps its whole output (up to TPW pixel tiles x FTW feature tiles) in accumulators, the
// workgroup waits until everybody has read the input map, and the output overwrites it.  Half the LDS of an input
// and an output map, so a tile holds twice the pixels with two workgroups per compute unit, and that is what the
// layer needs: with FTW = 2 feature tiles a wavefront's weight fragments (global, vector L1: 64 B/clk per compute
// unit) serve up to 9 pixel tiles instead of 4 or 5, and the halo that neighbouring strips recompute shrinks.
// Weight packing: A fragments [feature tile][chunk][lane][8], k = tap * C + ci.
//
// Measured, 1024 images, us, a section's two blocks together: 64 channels on 36 x 48 647 -> 584, 128 on 18 x 24 573 -> 474; 512
// images: 32 channels on 40 x 100 327 -> 268; 64 images: 16 on 60 x 400 173 -> 142; conv0 + pooling 64 -> 128 on 36 x 48 350 -> 296,
// 64 -> 64 on 18 x 24 61 -> 39; before: a cell as one 16-byte access per lane (the lanes of a feature tile pair fetch the
// packed weights' rows so that a lane's eight results are consecutive channels) instead of two of 8 bytes; border
// cells skipped, not rewritten with zeros; weights two chunks in registers, not three (at 128 registers to a wavefront the third
// spills now); no pointer picked at run time (its loads are flat ones and count as LDS traffic).  (The kernels
// that keep an input and an output map took 915 us for 64 channels on 36 x 48, 680 for 128 on 18 x 24.)
// What bounds them (64 channels on 36 x 48): HBM traffic 0.96 GB in the first block, 1.21 in the second (fp32 in), 155 and 190 us
// at the copy rate; the MFMAs take 119 us; about 5 K of the staging's 15 K cycles of a workgroup are bank conflicts of its
// writes.
#pragma once
#include "resnet_blockfused.h"

namespace seedinf {

constexpr int RS_THREADS = 512;
constexpr size_t RS_LDS_MAX = 80 * 1024;                    // two workgroups per compute unit

template <int C>
struct StripCfg {
    static_assert(C == 16 || C == 32 || C == 64 || C == 128, "widths with a strip kernel");
    static constexpr int NCG = C / 8, NFT = C / 16;
    static constexpr int FTW = C == 16 ? 1 : 2;             // feature tiles a wavefront multiplies with one map fragment
    static constexpr int NFG = NFT / FTW;
    static constexpr int NPG = 8 / NFG;                     // wavefronts (pixel groups) per feature group
    static constexpr int TPW = C == 16 ? 12 : 9;            // pixel tiles a wavefront's accumulators hold
    static constexpr int KCH = (9 * C + 31) / 32;
    static constexpr int MAX_TILES = TPW * NPG;
    // cells of a plane: `rows` rows and the right border of the last, in whole 256 bytes
    __host__ __device__ static constexpr int plane(int rows, int W) { return (rows * (W + 1) + 1 + 15) / 16 * 16; }
    static constexpr size_t lds_bytes(int rows, int W) { return (size_t)NCG * plane(rows, W) * 16; }
    __host__ __device__ static constexpr int tiles(int rows, int W) { return (rows * (W + 1) - 1 + 15) / 16; }
    static constexpr bool fits(int rows, int map_rows, int W)
    {
        return tiles(rows, W) <= MAX_TILES && lds_bytes(map_rows, W) <= RS_LDS_MAX;
    }
};

// logical workgroup of a launch: consecutive workgroups land on the eight XCDs in turn, so each XCD is given one run
// of consecutive strips, whose shared halo rows then meet in its L2
__device__ __forceinline__ int xcd_run(int idx, int total)
{
    const int per = total >> 3, rem = total & 7, x = idx & 7;
    return x * per + min(x, rem) + (idx >> 3);
}

// Zeroes a map's border cells: cell 0 of every row and the one behind the last row, the first and the last row where
// they lie outside the image.
template <int C>
__device__ __forceinline__ void zero_borders(char* map, int PL, int P, int rows, bool top, bool bottom, int tid)
{
    constexpr int NCG = C / 8, STEP = RS_THREADS / NCG;
    const bf16x8 z = {};
    char* plane = map + (tid % NCG) * PL * 16;
    for (int r = tid / NCG; r <= rows; r += STEP) *(bf16x8*)(plane + r * P * 16) = z;
    for (int c = tid / NCG; c < P; c += STEP) {
        if (top) *(bf16x8*)(plane + c * 16) = z;
        if (bottom) *(bf16x8*)(plane + ((rows - 1) * P + c) * 16) = z;
    }
}

// The lane number, worked out afresh: what follows from it is not hoisted over (and spilled across) the phases.
__device__ __forceinline__ int fresh_lane(int lane)
{
    asm volatile("" : "+v"(lane));
    return lane;
}

// Pixel tiles whose map fragments strip_conv keeps requested ahead: divides NT so that a slot serves the same tiles in every chunk.
constexpr int strip_ring(int NT) { return NT % 4 == 0 ? 4 : (NT % 3 == 0 ? 3 : (NT % 5 == 0 ? 5 : NT)); }

// A wavefront's weight fragments: WS slots, requested WS - 1 chunks ahead.
// With two feature tiles (FTW = 2) the two fragments together hold, for lane group g of the result, the eight consecutive
// channels 8 g .. 8 g + 7 of the pair's 32 instead of four of each tile: the lanes fetch the rows of the packed weights in
// that order.
template <int C, int WS = 2>
struct StripWeights {
    using K = StripCfg<C>;
    static constexpr int FTW = K::FTW, KCH = K::KCH, WJ = 4;
    bf16x8 a[WS][FTW];
    __device__ static __forceinline__ int first(int lane)
    {
        return FTW == 2 ? ((lane & 8) >> 3) * KCH * 64 + (lane & 48) + (lane & 4) * 2 + (lane & 3) : lane;
    }
    __device__ __forceinline__ void request(const bf16x8* __restrict__ wl, int kc, int slot, int lane)
    {
#pragma unroll
        for (int j = 0; j < FTW; ++j) a[slot][j] = (wl + j * WJ + kc * 64)[first(lane)];
    }
    // the first WS - 1 chunks
    __device__ __forceinline__ void start(const bf16x8* __restrict__ wl, int lane)
    {
#pragma unroll
        for (int d = 0; d < WS - 1; ++d) request(wl, d, d, lane);
    }
};

// acc[i][j] = convolution of pixel tile pg + NPG * i and feature tile ft0 + j of a region that starts at `src` (tap
// (0, 0) of its first pixel, plane 0): pixel q has tap (kh, kw) at cell q + kh * P + kw.  `last`: the region's last
// pixel, which lanes past the end read again.  The weights' first chunks have been requested (start); tail() runs
// behind the request of the last ones.
template <int C, int NT, int RING, int WS, class Tail>
__device__ __forceinline__ void strip_conv(const char* src, int PL, int P, int pg, int last, const bf16x8* __restrict__ wl, int lane,
                                           StripWeights<C, WS>& w, floatx4 (&acc)[NT][StripCfg<C>::FTW], Tail tail)
{
    using K = StripCfg<C>;
    constexpr int FTW = K::FTW, KCH = K::KCH, STEP = K::NPG * 256;
    static_assert(NT % RING == 0, "a ring slot's tiles");
    // Map fragments travel in a ring of RING registers sets, RING tiles (of this chunk or the next) ahead of their use.
    // The order is pinned: left alone, the compiler saves registers by asking for every fragment right before its MFMAs,
    // and each then waits out an LDS trip (64 channels on 36 x 48, 1024 images: 361 us).
    lane = fresh_lane(lane);
    const int g = lane >> 4, n = lane & 15;
    const int q0 = pg * 16 + n, ql = min(q0 + (NT - 1) * K::NPG * 16, last);
    const int plane = (C == 16 ? (g & 1) : g) * PL;
    const char* s0 = src + (plane + min(q0, last)) * 16;
    const char* sl = src + (plane + ql) * 16;
    // byte offset of chunk kc's tap and channel planes
    auto off = [&](int kc) {
        if constexpr (C == 16) {
            const int t0 = 2 * kc, t1 = min(2 * kc + 1, 8);  // (the tenth tap has zero weights)
            const int o0 = (t0 / 3) * P + t0 % 3, o1 = (t1 / 3) * P + t1 % 3;
            return ((g >> 1) ? o1 : o0) * 16;
        } else {
            constexpr int CPT = C / 32;
            const int tap = kc / CPT;
            return ((kc % CPT) * 4 * PL + (tap / 3) * P + tap % 3) * 16;
        }
    };
    auto frag = [&](int o, int i) { return *(const bf16x8*)((i < NT - 1 ? s0 + i * STEP : sl) + o); };
    bf16x8 b[RING];
    int o = off(0);
#pragma unroll
    for (int i = 0; i < RING; ++i) b[i] = frag(o, i);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < FTW; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // chunk kc, its weights in slot D; MORE: weights are left to request, NEXT: another chunk follows
    auto chunk = [&](int kc, auto dc, auto more, auto next) {
        constexpr int D = decltype(dc)::value;
        constexpr bool MORE = decltype(more)::value, NEXT = decltype(next)::value;
        const int on = NEXT ? off(kc + 1) : 0;
        if constexpr (MORE) w.request(wl, kc + WS - 1, (D + WS - 1) % WS, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
#pragma unroll
            for (int j = 0; j < FTW; ++j) acc[i][j] = mfma16(w.a[D][j], b[i % RING], acc[i][j]);
            if (i + RING < NT) b[i % RING] = frag(o, i + RING);
            else if constexpr (NEXT) b[i % RING] = frag(on, i + RING - NT);
            __builtin_amdgcn_sched_barrier(0);
        }
        o = on;
    };
    using D0 = std::integral_constant<int, 0>; using D1 = std::integral_constant<int, 1>; using D2 = std::integral_constant<int, 2>;
    using T = std::true_type; using F = std::false_type;
    constexpr int LEFT = KCH % WS == 0 ? WS : KCH % WS;      // chunks behind the loop
    static_assert(LEFT <= WS && (WS == 2 || KCH % WS == 0), "the last groups below");
#pragma unroll 1
    for (int kc = 0; kc < KCH - LEFT; kc += WS) {
        chunk(kc, D0{}, T{}, T{});
        chunk(kc + 1, D1{}, T{}, T{});
        if constexpr (WS == 3) chunk(kc + 2, D2{}, T{}, T{});
    }
    if constexpr (LEFT == 3) {
        chunk(KCH - 3, D0{}, T{}, T{});
        tail();
        chunk(KCH - 2, D1{}, F{}, T{});
        chunk(KCH - 1, D2{}, F{}, F{});
    } else if constexpr (LEFT == 2) {
        chunk(KCH - 2, D0{}, T{}, T{});
        tail();
        chunk(KCH - 1, D1{}, F{}, F{});
    } else {
        tail();
        chunk(KCH - 1, D0{}, F{}, F{});
    }
}
// Calls phase(NT) for the number of pixel tiles this wavefront owns (uniform): a convolution and its epilogue with the
// count a constant.  (Barriers inside: every wavefront passes the same number of them whatever its count.  The plans give
// at most TPW; the clamp keeps a count beyond it from passing none.)
template <int TPW, class F>
__device__ __forceinline__ void by_tiles(int nt, F phase)
{
    static_assert(TPW <= 12, "a case for every count");
    auto go = [&](auto ntc) {
        if constexpr (decltype(ntc)::value <= TPW) phase(ntc);
    };
    switch (min(nt, TPW)) {
    case 0: go(std::integral_constant<int, 0>{}); break;
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    case 7: go(std::integral_constant<int, 7>{}); break;
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 9: go(std::integral_constant<int, 9>{}); break;
    case 10: go(std::integral_constant<int, 10>{}); break;
    case 11: go(std::integral_constant<int, 11>{}); break;
    case 12: go(std::integral_constant<int, 12>{}); break;
    }
}

// (row, column) of the lane's pixel in a wavefront's successive tiles, P cells to a row, step by step: all tiles'
// coordinates at once would need the registers the accumulators are in.
struct TileWalk {
    int q, r, c, dr, dc, P, step;
    __device__ __forceinline__ TileWalk(int first, int step_, int P_) : q(first), P(P_), step(step_)
    {
        r = q / P; c = q - r * P;
        dr = step / P; dc = step - dr * P;
    }
    __device__ __forceinline__ void next()
    {
        q += step; c += dc; r += dr;
        if (c >= P) { c -= P; ++r; }
    }
};

// ---- residual blocks ----------------------------------------------------------
struct StripBlockArgs {
    const void* x_in;                  // [B, H, W, C]: bf16 (first block: the pooled map, whose values are bf16 by origin) or fp32
    const bf16x8* wp[2];               // conv_a, conv_b
    const float* bias[2];
    float* x_out;                      // first block: fp32 x' [B, H, W, C]
    __bf16* y;                         // second block
    int y_relu, ldy;                   // rectify y; ldy > 0: y is the feature matrix [B, ldy], (h, w, c) order
    int B, H, W, TH, strips, groups;   // strips of TH rows per image; workgroups
};

struct StripBlockPlan {
    int TH = 0, strips = 0;            // TH == 0: no strip fits
    long cells = 0;                    // map cells the two convolutions of a block walk over all strips
    // Rows per strip: the cut with the least work (tiles per wavefront, both convolutions, the halo row that
    // conv_a computes on each inner side included) that fits.
    template <int C>
    bool choose(int H, int W)
    {
        using K = StripCfg<C>;
        long best = -1;
        for (int ny = 1; ny <= H; ++ny) {
            const int th = (H + ny - 1) / ny, ns = (H + th - 1) / th;
            const int ra = conv_a_rows(th, ns);
            if (!K::fits(ra, ra + 2, W)) continue;
            const long tiles = (long)ns * (K::tiles(ra, W) + K::tiles(th, W)), cost = tiles + (long)ns * 2 * K::NPG;
            if (best < 0 || cost < best) { best = cost; TH = th; strips = ns; cells = tiles * 16; }
        }
        return best >= 0;
    }
    static int conv_a_rows(int th, int ns) { return ns == 1 ? th : (ns == 2 ? th + 1 : th + 2); }
};

// FIRST: bf16 in, fp32 out; else fp32 in, bf16 out.
template <int C, bool FIRST>
__global__ __launch_bounds__(RS_THREADS, 4) void strip_block_kernel(StripBlockArgs p)
{
    using K = StripCfg<C>;
    constexpr int FTW = K::FTW, TPW = K::TPW, CPL = 4 * FTW;      // a lane's channels of a pixel
    typedef __bf16 lane_bf16 __attribute__((ext_vector_type(CPL)));
    extern __shared__ __attribute__((aligned(16))) char rs_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = xcd_run(blockIdx.x, p.groups);
    const int P = p.W + 1;
    const int b = wg / p.strips;
    const int y0 = (wg % p.strips) * p.TH;
    const int ye = min(y0 + p.TH, p.H);                      // the strip's rows: y0 .. ye - 1
    // map row 0 is image row m0; conv_a covers image rows ya .. yz - 1, conv_b the strip's
    const int m0 = max(y0 - 2, -1), ya = max(y0 - 1, 0), yz = min(ye + 1, p.H);
    const int arow = ya - m0, brow = y0 - m0;
    const int ra = yz - ya, rb = ye - y0;
    const int MR = arow + ra + 1;
    const int PL = K::plane(MR, p.W);
    const size_t img = (size_t)p.H * p.W * C;

    // ---- R = ReLU(x) as bf16 ----
    // The strip's pixels are one run of memory, so an item's address is a running offset and
    // only its cell needs a (row, column) walk; the border cells are zeroed apart (walked cell by cell with the border in
    // it, the loop spent 25 K cycles of a workgroup against 15 K: 64 channels on 36 x 48, 334 -> 310 us).  All of a
    // thread's loads, or half of them in fp32, are requested before the first conversion.
    {
        constexpr int UNR = FIRST ? 10 : 5, CSTEP = RS_THREADS / K::NCG, EB = FIRST ? 2 : 4;
        static_assert(RS_THREADS % K::NCG == 0, "a thread keeps its channel group");
        const int cg = tid % K::NCG;
        const int t0 = max(m0, 0), t1 = min(m0 + MR, p.H);      // image rows in the map
        const int npx = (t1 - t0) * p.W;
        const char* src = (const char*)p.x_in + (b * img + (size_t)t0 * p.W * C) * EB;
        zero_borders<C>(rs_lds, PL, P, MR, m0 < 0, m0 + MR > p.H, tid);
        RowWalk rw(tid / K::NCG, CSTEP, p.W);
        int px = tid / K::NCG;
        uint32_t from = (uint32_t)(px * C + cg * 8) * EB;
        char* const plane = rs_lds + (cg * PL + (t0 - m0) * P + 1) * 16;
        for (; px < npx; px += UNR * CSTEP) {
            floatx4 lo[UNR], hi[UNR];
            bf16x8 v[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u, from += CSTEP * C * EB) {
                if (px + u * CSTEP >= npx) continue;
                if constexpr (FIRST) {
                    v[u] = *(const bf16x8*)(src + from);
                } else {
                    lo[u] = *(const floatx4*)(src + from);
                    hi[u] = *(const floatx4*)(src + from + 16);
                }
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                char* cell = plane + (rw.r * P + rw.c) * 16;
                rw.next();
                if (px + u * CSTEP >= npx) continue;
                const bf16x8 raw = FIRST ? v[u] : to_bf16x8(lo[u], hi[u]);
                const bf16x4 l = relu_bf16x4(__builtin_shufflevector(raw, raw, 0, 1, 2, 3));
                const bf16x4 h = relu_bf16x4(__builtin_shufflevector(raw, raw, 4, 5, 6, 7));
                *(bf16x8*)cell = __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
    }
    __syncthreads();

    const int fg = wave % K::NFG, pg = wave / K::NFG;
    auto tiles_of = [&](int npix) { return ((npix + 15) / 16 - pg + K::NPG - 1) / K::NPG; };      // (at most TPW: the host's plan)
    auto convolve = [&](int conv, int row, int np, auto& acc, auto ntc) {
        constexpr int NT = decltype(ntc)::value;
        const bf16x8* const wl = p.wp[conv] + fg * FTW * K::KCH * 64;
        StripWeights<C> w;
        w.start(wl, fresh_lane(lane));
        strip_conv<C, NT, strip_ring(NT)>(rs_lds + (row - 1) * P * 16, PL, P, pg, np - 1, wl, lane, w, acc, [] {});
    };
    auto join = [](const bf16x4 (&r)[FTW]) {
        if constexpr (FTW == 2) return __builtin_shufflevector(r[0], r[1], 0, 1, 2, 3, 4, 5, 6, 7);
        else return r[0];
    };
    // ---- U = ReLU(conv_a(R) + bias), in place (border cells keep their zeros) ----
    const int npa = ra * P - 1;
    by_tiles<TPW>(tiles_of(npa), [&](auto ntc) {
        constexpr int NT = decltype(ntc)::value;
        if constexpr (NT == 0) {
            __syncthreads();
        } else {
            floatx4 acc[NT][FTW];
            convolve(0, arow, npa, acc, ntc);
            const int ln = fresh_lane(lane), g = ln >> 4;
            floatx4 bv[FTW];
#pragma unroll
            for (int j = 0; j < FTW; ++j) bv[j] = *(const floatx4*)(p.bias[0] + fg * FTW * 16 + g * CPL + j * 4);
            __syncthreads();                                 // everybody has read R
            TileWalk w(pg * 16 + (ln & 15), K::NPG * 16, P);
            char* cell = rs_lds + (arow * P + 1 + w.q) * 16 + (FTW == 2 ? (fg * 4 + g) * PL * 16 : (g >> 1) * PL * 16 + (g & 1) * 8);
#pragma unroll
            for (int i = 0; i < NT; ++i, w.next(), cell += K::NPG * 256) {
                bf16x4 r[FTW];
#pragma unroll
                for (int j = 0; j < FTW; ++j) r[j] = relu_bf16x4(to_bf16x4(acc[i][j] + bv[j]));
                if (w.c < p.W && (i < NT - 1 || w.q < npa)) *(lane_bf16*)cell = join(r);
            }
        }
    });
    __syncthreads();
    // ---- x' = x + conv_b(U) + bias ----
    const int npb = rb * P - 1;
    by_tiles<TPW>(tiles_of(npb), [&](auto ntc) {
        constexpr int NT = decltype(ntc)::value;
        if constexpr (NT > 0) {
            floatx4 acc[NT][FTW];
            convolve(1, brow, npb, acc, ntc);
            const int ln = fresh_lane(lane), g = ln >> 4;
            const int f0 = fg * FTW * 16 + g * CPL;
            floatx4 bv[FTW];
#pragma unroll
            for (int j = 0; j < FTW; ++j) bv[j] = *(const floatx4*)(p.bias[1] + f0 + j * 4);
            TileWalk w(pg * 16 + (ln & 15), K::NPG * 16, P);
            // residuals are requested XB tiles ahead of their use: one tile at a time, each waits out a trip to memory
            constexpr int XB = C == 16 ? 4 : 2;
            lane_bf16 rb16[XB];
            floatx4 r32[XB][FTW];
            int at[XB];                                      // element offset from the image; -1: no pixel
            auto request = [&](int i) {
                at[i % XB] = w.c < p.W && (i < NT - 1 || w.q < npb) ? ((y0 + w.r) * p.W + w.c) * C + f0 : -1;
                w.next();
                const int from = max(at[i % XB], 0);
                if constexpr (FIRST) {
                    rb16[i % XB] = *(const lane_bf16*)((const __bf16*)p.x_in + b * img + from);
                } else {
#pragma unroll
                    for (int j = 0; j < FTW; ++j) r32[i % XB][j] = *(const floatx4*)((const float*)p.x_in + b * img + from + j * 4);
                }
            };
#pragma unroll
            for (int i = 0; i < XB && i < NT; ++i) request(i);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int u = i % XB;
                if (at[u] >= 0) {
                    bf16x4 t[FTW];
#pragma unroll
                    for (int j = 0; j < FTW; ++j) {
                        floatx4 v = acc[i][j] + bv[j];
                        if constexpr (FIRST) {
                            const bf16x4 x = j == 0 ? __builtin_shufflevector(rb16[u], rb16[u], 0, 1, 2, 3)
                                                    : __builtin_shufflevector(rb16[u], rb16[u], CPL - 4, CPL - 3, CPL - 2, CPL - 1);
                            v += to_floatx4(x);
                            *(floatx4*)(p.x_out + b * img + at[u] + j * 4) = v;
                        } else {
                            v += r32[u][j];
                            t[j] = to_bf16x4(v);
                            if (p.y_relu) t[j] = relu_bf16x4(t[j]);
                        }
                    }
                    if constexpr (!FIRST) *(lane_bf16*)(p.y + (p.ldy > 0 ? (size_t)b * p.ldy : b * img) + at[u]) = join(t);
                }
                if (i + XB < NT) request(i + XB);
            }
        }
    });
}

// ---- conv0 of a later section with its pooling --------------------------------
// bf16 NHWC input of C channels -> 3x3 SAME convolution -> 3x3 / stride-2 max-pool -> the section's x as bf16 (the
// maxima of values that were rounded to bf16 before they were compared: no rounding of its own).  A workgroup
// computes C of the layer's output channels (neighbouring workgroups: the others), so that its output fits over its input, for the
// convolution rows under PTH pooled rows; window cells outside the map are clamped onto it.
struct StripPoolArgs {
    const __bf16* in;                  // [B, H, W, C]
    const bf16x8* wp;                  // [COUT / 16][chunks][64 lanes][8], k = tap * C + ci
    const float* bias;
    __bf16* x;                         // [B, PH, PW, COUT]
    int B, H, W, PH, PW, pad_h, pad_w, COUT, PTH, strips, groups;
};

struct StripPoolPlan {
    int PTH = 0, strips = 0, rows = 0; // PTH == 0: no strip fits; rows: the most convolution rows a strip covers
    template <int C>
    bool choose(int H, int W, int PH, int pad_h)
    {
        using K = StripCfg<C>;
        long best = -1;
        for (int pth = 1; pth <= PH; ++pth) {
            const int ns = (PH + pth - 1) / pth;
            int r = 0;
            long work = 0;
            for (int s = 0; s < ns; ++s) {
                const int p0 = s * pth, p1 = std::min(p0 + pth, PH);
                const int n = std::min(2 * (p1 - 1) - pad_h + 2, H - 1) - std::max(2 * p0 - pad_h, 0) + 1;
                r = std::max(r, n);
                work += K::tiles(n, W) + 2 * K::NPG;
            }
            if (!K::fits(r, r + 2, W)) continue;
            if (best < 0 || work < best) { best = work; PTH = pth; strips = ns; rows = r; }
        }
        return best >= 0;
    }
};

template <int C>
__global__ __launch_bounds__(RS_THREADS, 4) void strip_pool_kernel(StripPoolArgs p)
{
    using K = StripCfg<C>;
    constexpr int FTW = K::FTW, TPW = K::TPW;
    extern __shared__ __attribute__((aligned(16))) char rs_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n = lane & 15;
    // the feature groups of a strip are neighbours: they read the same input
    const int nf = p.COUT / C;
    const int wg = xcd_run(blockIdx.x, p.groups);
    const int fbase = (wg % nf) * K::NFT, strip = wg / nf;
    const int b = strip / p.strips, ph0 = (strip % p.strips) * p.PTH, ph1 = min(ph0 + p.PTH, p.PH);
    const int P = p.W + 1;
    const int yc = max(2 * ph0 - p.pad_h, 0), yz = min(2 * (ph1 - 1) - p.pad_h + 3, p.H);      // convolution rows yc .. yz - 1
    const int m0 = yc - 1, rows = yz - yc, MR = rows + 2;
    const int PL = K::plane(MR, p.W);
    {
        constexpr int UNR = 10, CSTEP = RS_THREADS / K::NCG;
        const int cg = tid % K::NCG;
        const int t0 = max(m0, 0), t1 = min(m0 + MR, p.H), npx = (t1 - t0) * p.W;
        const char* src = (const char*)(p.in + ((size_t)b * p.H + t0) * p.W * C);
        zero_borders<C>(rs_lds, PL, P, MR, m0 < 0, m0 + MR > p.H, tid);
        RowWalk rw(tid / K::NCG, CSTEP, p.W);
        int px = tid / K::NCG;
        uint32_t from = (uint32_t)(px * C + cg * 8) * 2;
        char* const plane = rs_lds + (cg * PL + (t0 - m0) * P + 1) * 16;
        for (; px < npx; px += UNR * CSTEP) {
            bf16x8 v[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u, from += CSTEP * C * 2)
                if (px + u * CSTEP < npx) v[u] = *(const bf16x8*)(src + from);
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                char* cell = plane + (rw.r * P + rw.c) * 16;
                rw.next();
                if (px + u * CSTEP < npx) *(bf16x8*)cell = v[u];
            }
        }
    }
    __syncthreads();

    {
        const int fg = wave % K::NFG, pg = wave / K::NFG;
        const int ft0 = fg * FTW;
        const int npix = rows * P - 1;
        by_tiles<TPW>(((npix + 15) / 16 - pg + K::NPG - 1) / K::NPG, [&](auto ntc) {
            constexpr int NT = decltype(ntc)::value;
            if constexpr (NT == 0) {
                __syncthreads();
            } else {
                floatx4 acc[NT][FTW];
                const bf16x8* const wl = p.wp + (size_t)(fbase + ft0) * K::KCH * 64;
                StripWeights<C> w;
                w.start(wl, fresh_lane(lane));
                strip_conv<C, NT, strip_ring(NT)>(rs_lds, PL, P, pg, npix - 1, wl, lane, w, acc, [] {});
                floatx4 bv[FTW];
#pragma unroll
                for (int j = 0; j < FTW; ++j) bv[j] = *(const floatx4*)(p.bias + (fbase + ft0) * 16 + g * 4 * FTW + j * 4);
                __syncthreads();                             // everybody has read the input
                char* cell = rs_lds + (P + 1 + pg * 16 + n) * 16 + (FTW == 2 ? (fg * 4 + g) * PL * 16 : (g >> 1) * PL * 16 + (g & 1) * 8);
#pragma unroll
                for (int i = 0; i < NT; ++i, cell += K::NPG * 256) {
                    if (i == NT - 1 && (pg + K::NPG * i) * 16 + n >= npix) continue;
                    bf16x4 r[FTW];
#pragma unroll
                    for (int j = 0; j < FTW; ++j) r[j] = to_bf16x4(acc[i][j] + bv[j]);
                    if constexpr (FTW == 2) *(bf16x8*)cell = __builtin_shufflevector(r[0], r[1], 0, 1, 2, 3, 4, 5, 6, 7);
                    else *(bf16x4*)cell = r[0];
                }
            }
        });
    }
    __syncthreads();

    // a wavefront pools PXW consecutive pixels x CGW channel groups at a time: reads of one plane are two cells apart
    constexpr int CGW = K::NCG < 8 ? K::NCG : 8, PXW = 64 / CGW, NCB = K::NCG / CGW;
    const int pxl = lane % PXW, cgl = lane / PXW;
    const int npool = (ph1 - ph0) * p.PW;
    for (int it = wave; it < (npool + PXW - 1) / PXW * NCB; it += RS_THREADS / 64) {
        const int px = (it / NCB) * PXW + pxl, cg = (it % NCB) * CGW + cgl;
        if (px >= npool) continue;
        const int ph = px / p.PW, pw = px - ph * p.PW;
        const int y = 2 * (ph0 + ph) - p.pad_h, x = 2 * pw - p.pad_w;
        const char* pl = rs_lds + (size_t)(cg * PL + 1) * 16;
        uint4 m;
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
            const char* row = pl + (size_t)((min(max(y + dy, yc), yz - 1) - m0) * P) * 16;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const uint4 v = *(const uint4*)(row + min(max(x + dx, 0), p.W - 1) * 16);
                m = dy + dx == 0 ? v : bf16x8_max(m, v);
            }
        }
        *(uint4*)(p.x + (((size_t)b * p.PH + ph0 + ph) * p.PW + pw) * p.COUT + fbase * 16 + cg * 8) = m;
    }
}

}  // namespace seedinf
