// The dense comparator of Section 3.1 on bf16 operands: nothing is lowered in memory.
//
//   out[k][y*Ow + x] = sum over (c, l, w) of W[k][(c*kh + l)*kw + w] * padded input(c, y*stride + l, x*stride + w)
//
// A workgroup owns 32 * TM * wm kernels x 32 * TN * wn positions; its groups of wm x wn wavefronts take
// the chunks of sixteen input channels in turn.  A group brings a chunk's window (the input cells behind
// its positions, bias and ReLU of a producing layer applied, rounded to nearest-even bf16) into LDS with the
// channels innermost, so that for one kernel cell a lane's operand of v_mfma_f32_32x32x16_bf16 - eight
// channels at one position - is one 16-byte read, the kernel cell a scalar offset.  The next chunk's window
// is on its way (two LDS buffers, one barrier per chunk) while the matrix cores work.  The weights' operands
// come from memory straight into registers, three steps ahead: reorder_weights_kernel has put them in the
// order of use (chunk, kernel cell, half of the channels, kernel), which costs one short launch.
//
// Lowering in memory moved 18 bytes per input cell of a 3x3 layer out and back in.
#include "conv_tiles.hpp"

#include <cmath>
#include <utility>

namespace cpoconv {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// two floats -> two bf16, round to nearest even (v_cvt_pk_bf16_f32), low half first
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const floatx2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// ---- the kernel matrix -----------------------------------------------------------------------------

// The kernel matrix K x Kd (fp32, row-major) in groups of eight consecutive contraction indices:
// [ceil(Kd/8)][round_up(K,64)][8], rounded to nearest-even bf16, zero filled.
__global__ __launch_bounds__(256) void prepare_weights_bf16_kernel(const float *__restrict__ w, uint16_t *__restrict__ wb,
                                                                  const int M, const int Mp, const int Kd, const int K8)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;   // one 16-byte group: (k8, m)
    if (idx >= K8 * Mp) return;
    const int k8 = idx / Mp, m = idx - k8 * Mp;
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int k = 8 * k8 + u;
        v[u] = (m < M && k < Kd) ? w[static_cast<int64_t>(m) * Kd + k] : 0.0f;
    }
    reinterpret_cast<uint4 *>(wb)[idx] = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]),
                                                    pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
}

// The same matrix in the order of use: [chunk of 16 channels][kernel cell][channels 0 - 7, 8 - 15][round_up(K,64)][8],
// from the groups above (kPrepared) or from fp32.  A thread writes one group of 16 bytes.
template <bool kPrepared>
__global__ __launch_bounds__(256) void reorder_weights_kernel(const void *__restrict__ w, uint4 *__restrict__ ordered, const int M,
                                                             const int Mp, const int C, const int taps, const int64_t groups)
{
    const int64_t idx = blockIdx.x * int64_t{256} + threadIdx.x;
    if (idx >= groups) return;
    const int64_t row = idx / Mp;   // (chunk, cell, half)
    const int m = static_cast<int>(idx - row * Mp), half = row & 1, step = static_cast<int>(row >> 1);
    const int chunk = step / taps, tap = step - chunk * taps;
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int c = chunk * 16 + half * 8 + u;
        const int64_t q = static_cast<int64_t>(c) * taps + tap;
        if constexpr (kPrepared)
            v[u] = c < C ? static_cast<const uint16_t *>(w)[((q >> 3) * Mp + m) * 8 + (q & 7)] : 0;
        else
            v[u] = pack_bf16(c < C && m < M ? static_cast<const float *>(w)[static_cast<int64_t>(m) * C * taps + q] : 0.0f, 0.0f);
    }
    ordered[idx] = make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
}

int64_t ordered_groups(const Geometry &g) { return (g.C + 15) / 16 * int64_t{2} * g.kh * g.kw * g.Kpad; }

// ---- the convolution -------------------------------------------------------------------------------

struct Bf16Args {
    int32_t C, K, Kpad, N;
    int32_t H, W, pad_h, pad_w;
    int32_t Ih, Iw, Oh, Ow, stride, kw, taps;
    int32_t SW, cols, cells;           // strip width in outputs; window extent behind a tile
    int32_t nchunks;                   // chunks of sixteen channels
    int32_t tiles, per_m;              // tiles of a strip, of all strips
    int32_t wm, wn, groups;            // wavefronts of a group over kernels and positions, groups
    int32_t window_bytes, buffers;     // LDS: one or two windows per group
    int32_t relu;
    Divisor by_SW, by_Oh, by_Ih, by_cols, by_tiles, by_per_m;
    int64_t map_image;
    int32_t map_c, map_r, map_x;       // strides of the map
    const float *values;
    const float *bias;
    const uint4 *weights;
    float *out;
};

__host__ __device__ constexpr int max_waves(int tm, int) { return tm >= 2 ? 8 : 16; }

template <typename Step, int... d>
__device__ __forceinline__ void steps(const Step &step, int next, std::integer_sequence<int, d...>)
{
    (step(std::integral_constant<int, d>(), next + d), ...);
}

// kTaps: kernel cells, where the instantiation knows them (0: any number)
template <int TM, int TN, int kTaps, bool kFar>
__global__ __launch_bounds__(64 * max_waves(TM, TN)) void conv_bf16_kernel(const Bf16Args a)
{
    typedef Buffer<kFar> Array;
    typedef typename Array::Offset Offset;
    // Steps whose weights have registers.  Loads complete in order, so a weight loaded behind the next
    // window's loads waits for them: with a whole chunk's weights in registers every load has the time of a
    // chunk to arrive.
    constexpr int D = kTaps != 0 && kTaps <= 9 ? kTaps : (kTaps != 0 && kTaps % 5 == 0 ? 5 : 4);
    constexpr int IT = 2;   // window pieces (eight channels of a cell) a thread holds on their way
    extern __shared__ __align__(16) char smem[];
    const int lane = lane_id(), n = lane & 31, half = lane >> 5;
    const int wave = uni(threadIdx.x / kLanes), team = a.wm * a.wn;
    const int group = wave / team, in_group = wave - group * team, wn = in_group / a.wm, wm = in_group - wn * a.wm;
    const int thread = in_group * kLanes + lane, threads = team * kLanes;

    const int number = dealt(blockIdx.x, gridDim.x);
    const int mb = quotient(number, a.by_per_m), in_m = number - mb * a.per_m;
    const int strip = quotient(in_m, a.by_tiles), tile = in_m - strip * a.tiles;
    const int kbase = (mb * a.wm + wm) * 32 * TM, p0 = tile * 32 * TN * a.wn, x0 = strip * a.SW;
    const int row0 = quotient(p0, a.by_SW), in_row0 = p0 - row0 * a.SW;
    const int image0 = quotient(row0, a.by_Oh), y0 = row0 - image0 * a.Oh, top = y0 * a.stride;
    const int positions = a.N * a.Oh * a.SW;

    // ---- the window's pieces: channels 0 - 7 of every cell, then 8 - 15 ---------------------------------
    const int pieces = 2 * a.cells;
    const int64_t channel_bytes = static_cast<int64_t>(a.map_c) * 4, image_bytes = a.map_image * 4;
    const char *source = reinterpret_cast<const char *>(a.values) + image0 * image_bytes;
    auto origin = [&](int i) __attribute__((always_inline)) {
        const int upper = i >= a.cells, cell = upper ? i - a.cells : i;
        const int r = quotient(cell, a.by_cols), q = cell - r * a.cols;
        const int v = top + r, image = quotient(v, a.by_Ih), hr = v - image * a.Ih - a.pad_h, jr = x0 * a.stride + q - a.pad_w;
        const bool ok = i < pieces && image0 + image < a.N && hr >= 0 && hr < a.H && jr >= 0 && jr < a.W;
        const Offset from = image * static_cast<Offset>(image_bytes) + static_cast<Offset>(hr) * (a.map_r * 4) +
                            static_cast<Offset>(jr) * (a.map_x * 4) + upper * static_cast<Offset>(8 * channel_bytes);
        return ok ? from : Array::kNothing;
    };
    auto load = [&](float (&x)[8], Offset from, int chunk) __attribute__((always_inline)) {
        const int64_t left = (a.N - image0) * image_bytes - chunk * (16 * channel_bytes);
        const Array buffer(source + chunk * (16 * channel_bytes), left > 0 ? left : 0);   // (past the last chunk: zeros)
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = buffer.load1(from, c * static_cast<Offset>(channel_bytes));
    };
    auto store = [&](char *window, float (&x)[8], Offset from, int i, int chunk) __attribute__((always_inline)) {
        const int c0 = chunk * 16 + (i >= a.cells ? 8 : 0);
        if (a.relu) {   // the end of the layer that produced the map; cells outside the map stay zero
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                if (a.bias != nullptr) x[c] += a.bias[min(c0 + c, a.C - 1)];
                x[c] = from != Array::kNothing && (__float_as_uint(x[c]) - 1u) < 0x7f800000u ? x[c] : 0.0f;
            }
        }
        if (chunk * 16 + 16 > a.C) {   // channels past the last one (the loads read on)
#pragma unroll
            for (int c = 0; c < 8; ++c) x[c] = c0 + c < a.C ? x[c] : 0.0f;
        }
        if (i < pieces)
            reinterpret_cast<uint4 *>(window)[i] = make_uint4(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7]));
    };
    Offset from[IT];
    float x[IT][8];
#pragma unroll
    for (int u = 0; u < IT; ++u) {
        from[u] = origin(thread + u * threads);
        load(x[u], from[u], group);
    }

    // ---- where the lane's positions and kernels start ---------------------------------------------------
    int base[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int in_tile = (wn * TN + t) * 32 + n, p = in_row0 + in_tile;
        const int row = quotient(p, a.by_SW), image = quotient(y0 + row, a.by_Oh);
        const int y = y0 + row - image * a.Oh, col = p - row * a.SW;
        const int cell = p0 + in_tile < positions ? (image * a.Ih + y * a.stride - top) * a.cols + col * a.stride : 0;
        base[t] = (half * a.cells + cell) * 16;
    }
    const Offset step_bytes = static_cast<Offset>(a.Kpad) * 32;
    const Array weights(a.weights, static_cast<int64_t>(a.nchunks) * a.taps * a.Kpad * 32);
    Offset at[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) at[m] = (static_cast<Offset>(half) * a.Kpad + min(kbase + m * 32, a.Kpad - 32) + n) * 16;
    uint4v w[D][TM];
    auto load_weights = [&](uint4v (&v)[TM], int step) __attribute__((always_inline)) {   // (past the end: zeros, not used)
#pragma unroll
        for (int m = 0; m < TM; ++m) v[m] = weights.load4(at[m], step * step_bytes);
    };

    floatx16 acc[TM][TN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[m][t][i] = 0.0f;

    // A group whose chunks have run out multiplies zeros.
    const int rounds = (a.nchunks + a.groups - 1) / a.groups;
    if constexpr (kTaps != 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) load_weights(w[d], group * kTaps + d);
    }
#pragma unroll 1
    for (int round = 0; round < rounds; ++round) {
        const int chunk = round * a.groups + group;
        char *window = smem + (group * a.buffers + (a.buffers == 2 ? round & 1 : 0)) * a.window_bytes;
        if (a.buffers == 1 && round > 0) __syncthreads();
#pragma unroll
        for (int u = 0; u < IT; ++u) store(window, x[u], from[u], thread + u * threads, chunk);
#pragma unroll 1
        for (int i = thread + IT * threads; i < pieces; i += threads) {
            const Offset o = origin(i);
            float more[8];
            load(more, o, chunk);
            store(window, more, o, i, chunk);
        }
        __syncthreads();
        if constexpr (kTaps == 0) {
#pragma unroll
            for (int d = 0; d < D - 1; ++d) load_weights(w[d], chunk * a.taps + d);
        }
#pragma unroll
        for (int u = 0; u < IT; ++u) load(x[u], from[u], chunk + a.groups);
        int offset = 0, column = 0;
        auto step_of = [&](auto d_, int next) __attribute__((always_inline)) {
            constexpr int d = decltype(d_)::value;
            uint4v b[TN];
#pragma unroll
            for (int t = 0; t < TN; ++t) b[t] = *reinterpret_cast<const uint4v *>(window + (base[t] + offset));
            offset += 16;
            if (++column == a.kw) {
                column = 0;
                offset += (a.cols - a.kw) * 16;
            }
#pragma unroll
            for (int m = 0; m < TM; ++m) asm volatile("" : "+v"(w[d][m]));   // complete from here on
            if constexpr (kTaps == 0) load_weights(w[(d + D - 1) % D], next);
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[d][m]), __builtin_bit_cast(bf16x8, b[t]),
                                                                        acc[m][t], 0, 0, 0);
            if constexpr (kTaps != 0) load_weights(w[d], next);
        };
        if constexpr (kTaps != 0) {
            // the ring goes on into the group's next chunk
#pragma unroll
            for (int tap0 = 0; tap0 < kTaps; tap0 += D) {
                const int ahead = tap0 + D < kTaps ? chunk * kTaps + tap0 + D : (chunk + a.groups) * kTaps;
                steps(step_of, ahead, std::make_integer_sequence<int, D>());
            }
        } else {
#pragma unroll 1
            for (int tap = 0; tap < a.taps; tap += D) {
                const int next = chunk * a.taps + tap + D - 1;
                step_of(std::integral_constant<int, 0>(), next);
                if (tap + 1 < a.taps) step_of(std::integral_constant<int, 1 % D>(), next + 1);
                if (tap + 2 < a.taps) step_of(std::integral_constant<int, 2 % D>(), next + 2);
                if (tap + 3 < a.taps) step_of(std::integral_constant<int, 3 % D>(), next + 3);
            }
        }
    }

    // ---- the groups' sums, added in group order; register i of a tile: kernel 8 * (i / 4) + 4 * half + i % 4 ----
    const int64_t plane = static_cast<int64_t>(a.Oh) * a.Ow;
    int64_t to[TN];
    bool ok[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int in_tile = (wn * TN + t) * 32 + n, p = in_row0 + in_tile;
        const int row = quotient(p, a.by_SW), image = quotient(y0 + row, a.by_Oh);
        const int y = y0 + row - image * a.Oh, col = x0 + p - row * a.SW;
        ok[t] = p0 + in_tile < positions && col < a.Ow;
        to[t] = (static_cast<int64_t>(image0 + image) * a.K + kbase + 4 * half) * plane + y * a.Ow + col;
    }
    const int left = a.K - kbase - 4 * half;
    if (a.groups == 1) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int k = m * 32 + 8 * (i >> 2) + (i & 3);
                    if (ok[t] && k < left) a.out[to[t] + k * plane] = acc[m][t][i];
                }
        return;
    }
    float *red = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int m = 0; m < TM; ++m) {   // tile by tile: 4 KB per wavefront
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 16; ++i) red[(wave * 16 + i) * kLanes + lane] = acc[m][t][i];
            __syncthreads();
            for (int i = group; i < 16; i += a.groups) {
                float s = red[(in_group * 16 + i) * kLanes + lane];
                for (int v = 1; v < a.groups; ++v) s += red[((v * team + in_group) * 16 + i) * kLanes + lane];
                const int k = m * 32 + 8 * (i >> 2) + (i & 3);
                if (ok[t] && k < left) a.out[to[t] + k * plane] = s;
            }
        }
}

// ---- launch shape ----------------------------------------------------------------------------------

struct Bf16Plan {
    int tm, tn, wm, wn, groups, sw;
    bool far, fits;
    int rows, cols, tiles, strips, mblocks, window_bytes, buffers, lds;
};

bool shape_plan(const Geometry &g, Bf16Plan *p)
{
    const int nb = 32 * p->tn * p->wn, taps = g.kh * g.kw;
    p->fits = false;
    p->rows = window_rows(g, nb, p->sw);
    p->cols = (p->sw - 1) * g.stride + g.kw;
    const int64_t cells = static_cast<int64_t>(p->rows) * p->cols, positions = static_cast<int64_t>(g.N) * g.Oh * p->sw;
    if (cells >= 65535 || positions >= (int64_t{1} << 31) - 4096) return false;
    const int64_t images = std::min<int64_t>(g.N, (nb - 1) / (static_cast<int64_t>(g.Oh) * p->sw) + 2), below = (int64_t{1} << 32) - 4096;
    p->far = 4 * images * g.C * g.H * g.W >= below || 16 * ordered_groups(g) + int64_t{20} * 64 * taps * g.Kpad >= below;
    if (p->far && p->tm * p->tn > 1) return false;
    p->tiles = static_cast<int>((positions + nb - 1) / nb);
    p->strips = (g.Ow + p->sw - 1) / p->sw;
    p->mblocks = (g.K + 32 * p->tm * p->wm - 1) / (32 * p->tm * p->wm);
    if (static_cast<int64_t>(p->tiles) * p->strips * p->mblocks >= (int64_t{1} << 31)) return false;
    const int nchunks = (g.C + 15) / 16, team = p->wm * p->wn;
    p->groups = std::min(std::min(p->groups, nchunks), max_waves(p->tm, p->tn) / team);
    p->groups = (nchunks + (nchunks + p->groups - 1) / p->groups - 1) / ((nchunks + p->groups - 1) / p->groups);
    p->window_bytes = static_cast<int>(cells) * 32;
    p->buffers = nchunks > p->groups ? 2 : 1;
    while (p->groups > 1 && p->groups * p->buffers * static_cast<int64_t>(p->window_bytes) > kLdsLimit) --p->groups;
    if (p->groups * p->buffers * static_cast<int64_t>(p->window_bytes) > kLdsLimit) p->buffers = 1;
    p->lds = std::max(p->groups * p->buffers * p->window_bytes, p->groups > 1 ? p->groups * team * 4096 : 0);
    p->fits = p->lds <= kLdsLimit;
    return p->fits;
}

// Estimated cycles: what a wavefront spends (matrix instructions of 32 cycles, the loads around them, its
// share of the windows), the load of the busiest compute unit, the latency of a lone workgroup, and the bytes
// of weights and windows a compute unit takes in.  The constants are fitted to 19 layers of 1 to 32 images x
// 30 to 360 launch shapes each, on MI355X: the shape picked is 3 % slower than the best one on average.
double plan_cost(const Geometry &g, const Bf16Plan &p)
{
    const int taps = g.kh * g.kw, nchunks = (g.C + 15) / 16, rounds = (nchunks + p.groups - 1) / p.groups;
    const int team = p.wm * p.wn, waves = p.groups * team, tiles = p.tm * p.tn, cells = p.rows * p.cols;
    const double step = tiles * 32.0 + 7.4 * p.tm + 0.6 * p.tn + 10.0;
    const double fill = (2 * cells + team * kLanes - 1) / (team * kLanes) * 243.0 + 702.0;
    const double wave = rounds * (taps * step + fill) + 121.0 + tiles * 718.0 * (p.groups > 1 ? 2.0 : 1.0);
    const double per_unit = static_cast<double>(p.tiles) * p.strips * p.mblocks / kComputeUnits;
    const double busiest = per_unit <= 6.0 ? std::ceil(per_unit) : per_unit;
    const double waves_per_simd = std::max(1.0, busiest * waves / 4.0);
    // wavefronts a SIMD holds, by the registers of the instantiations
    const bool whole = taps == 9 || taps == 25;
    const int simd = p.tm == 2 ? (p.tn == 2 ? (whole ? 2 : 3) : 4) : (p.tn == 2 && !whole && taps != 7 ? 5 : (p.tn == 2 ? 4 : 5));
    const int resident = std::max(1, std::min(4 * simd / waves, kLdsLimit / p.lds));
    const double active = std::min(resident * waves / 4.0, waves_per_simd);
    const double bytes = 32.0 * p.tm * p.wm * taps * 32.0 / 71.0 + cells * 64.0 / 137.0 * (1.0 + 300.0 / p.sw);
    const double through = waves_per_simd * wave * (1.0 + 0.58 / active) + busiest * nchunks * bytes;
    const double alone = rounds * (taps * (step + 529.0) + 348.0 + fill) + 121.0;
    return std::max(through, alone);
}

// The launch shape with the smallest estimate.  Strips: the whole width or an even part of it up to 64
// columns (whole lines of the map in one load), or eight or four columns (compact windows).
Bf16Plan bf16_plan(const Geometry &g)
{
    Bf16Plan best;
    best.fits = false;
    double least = 0.0;
    const int widths[] = {g.Ow, (g.Ow + 1) / 2, (g.Ow + 3) / 4, 8, 4};
    for (int tm : {2, 1})
        for (int tn : {2, 1})
            for (int wm : {1, 2, 4, 8})
                for (int wn : {1, 2, 4, 8})
                    for (int groups : {1, 2, 4, 8, 16}) {
                        if (wm * wn * groups > max_waves(tm, tn) || (tm * wm > 1 && 16 * tm * wm >= g.K) || (groups > 1 && 8 * groups >= g.C)) continue;
                        for (int sw : widths) {
                            if (sw > g.Ow || sw > 64) continue;
                            Bf16Plan p;
                            p.tm = tm; p.tn = tn; p.wm = wm; p.wn = wn; p.groups = groups; p.sw = sw;
                            if (!shape_plan(g, &p)) continue;
                            const double cost = plan_cost(g, p);
                            if (!best.fits || cost < least) {
                                best = p;
                                least = cost;
                            }
                        }
                    }
    if (!best.fits) {   // large strides: the least window there is
        best.tm = best.tn = best.wm = best.wn = best.groups = best.sw = 1;
        shape_plan(g, &best);
    }
    return best;
}

template <int TM, int TN>
void launch_kernel(const Bf16Plan &p, const Bf16Args &a, hipStream_t stream)
{
    const dim3 grid(p.tiles * p.strips * p.mblocks), block(p.groups * p.wm * p.wn * kLanes);
    switch (a.taps) {
    case 9: hipLaunchKernelGGL((conv_bf16_kernel<TM, TN, 9, false>), grid, block, p.lds, stream, a); break;
    case 7: hipLaunchKernelGGL((conv_bf16_kernel<TM, TN, 7, false>), grid, block, p.lds, stream, a); break;
    case 25: hipLaunchKernelGGL((conv_bf16_kernel<TM, TN, 25, false>), grid, block, p.lds, stream, a); break;
    default: hipLaunchKernelGGL((conv_bf16_kernel<TM, TN, 0, false>), grid, block, p.lds, stream, a);
    }
}

int launch(const Bf16Plan &p, const Geometry &g, const float *act, const Producer &prod, const uint4 *weights, float *out, hipStream_t stream)
{
    Bf16Args a = {};
    a.C = g.C; a.K = g.K; a.Kpad = g.Kpad; a.N = g.N;
    a.H = g.H; a.W = g.W; a.pad_h = g.pad_h; a.pad_w = g.pad_w;
    a.Ih = g.Ih; a.Iw = g.Iw; a.Oh = g.Oh; a.Ow = g.Ow; a.stride = g.stride; a.kw = g.kw; a.taps = g.kh * g.kw;
    a.SW = p.sw; a.cols = p.cols; a.cells = p.rows * p.cols;
    a.nchunks = (g.C + 15) / 16;
    a.tiles = p.tiles; a.per_m = p.tiles * p.strips;
    a.wm = p.wm; a.wn = p.wn; a.groups = p.groups;
    a.window_bytes = p.window_bytes; a.buffers = p.buffers;
    a.relu = prod.relu;
    a.by_SW = divisor(p.sw); a.by_Oh = divisor(g.Oh); a.by_Ih = divisor(g.Ih); a.by_cols = divisor(p.cols);
    a.by_tiles = divisor(p.tiles); a.by_per_m = divisor(a.per_m);
    a.map_image = static_cast<int64_t>(g.C) * g.H * g.W;
    a.map_c = g.channel_last ? 1 : g.H * g.W;
    a.map_r = g.channel_last ? g.W * g.C : g.W;
    a.map_x = g.channel_last ? g.C : 1;
    a.values = act;
    a.bias = prod.bias;
    a.weights = weights;
    a.out = out;
    KernelTimer timer("im2col_conv_bf16", stream);
    if (p.far)
        hipLaunchKernelGGL((conv_bf16_kernel<1, 1, 0, true>), dim3(p.tiles * p.strips * p.mblocks), dim3(p.groups * p.wm * p.wn * kLanes), p.lds,
                           stream, a);
    else if (p.tm == 2 && p.tn == 2) launch_kernel<2, 2>(p, a, stream);
    else if (p.tm == 2 && p.tn == 1) launch_kernel<2, 1>(p, a, stream);
    else if (p.tm == 1 && p.tn == 2) launch_kernel<1, 2>(p, a, stream);
    else launch_kernel<1, 1>(p, a, stream);
    CPOCONV_HIP_TRY(hipGetLastError());
    return CPOCONV_OK;
}

const Bf16Plan &cached_plan(const Geometry &g)
{
    struct Key {
        int32_t C, H, W, K, kh, kw, stride, pad_h, pad_w, N;
    };
    static thread_local ShapeCache<Key, Bf16Plan, 64> cache;
    const Key key = {g.C, g.H, g.W, g.K, g.kh, g.kw, g.stride, g.pad_h, g.pad_w, g.N};
    return cache.get(key, [&](Bf16Plan &p) { p = bf16_plan(g); });
}

}  // namespace

int64_t im2col_weights_bf16_len(const Geometry &g)
{
    return (static_cast<int64_t>(g.C) * g.kh * g.kw + 7) / 8 * g.Kpad * 8;
}

int64_t im2col_scratch_bytes(const Geometry &g)
{
    // what a lowered matrix takes as the paper counts it (four bytes an entry); the bf16 calls keep their
    // reordered kernel matrix here
    const int64_t lowered = static_cast<int64_t>(g.N) * g.C * g.kh * g.kw * g.Oh * g.Ow * 4;
    return (std::max(lowered, 16 * ordered_groups(g)) + 255) / 256 * 256;
}

int launch_prepare_weights_bf16(const float *w, const Geometry &g, uint16_t *wb, hipStream_t stream)
{
    const int Kd = g.C * g.kh * g.kw, K8 = (Kd + 7) / 8;
    KernelTimer timer("prepare_weights_bf16", stream);
    hipLaunchKernelGGL(prepare_weights_bf16_kernel, dim3((K8 * g.Kpad + 255) / 256), dim3(256), 0, stream, w, wb, g.K, g.Kpad, Kd, K8);
    CPOCONV_HIP_TRY(hipGetLastError());
    return CPOCONV_OK;
}

int launch_im2col_conv(const float *act, const Producer &prod, const Geometry &g, const void *w, void *scratch, float *out,
                       int precision, hipStream_t stream)
{
    if (precision == 0) return launch_conv_dense_f32(act, prod, g, static_cast<const float *>(w), out, stream);
    uint4 *ordered = static_cast<uint4 *>(scratch);
    const int64_t groups = ordered_groups(g);
    {
        KernelTimer timer("reorder_weights", stream);
        const dim3 grid(static_cast<unsigned>((groups + 255) / 256));
        if (precision == 2)
            hipLaunchKernelGGL(reorder_weights_kernel<true>, grid, dim3(256), 0, stream, w, ordered, g.K, g.Kpad, g.C, g.kh * g.kw, groups);
        else
            hipLaunchKernelGGL(reorder_weights_kernel<false>, grid, dim3(256), 0, stream, w, ordered, g.K, g.Kpad, g.C, g.kh * g.kw, groups);
        CPOCONV_HIP_TRY(hipGetLastError());
    }
    const Bf16Plan &p = cached_plan(g);
    if (p.fits) return launch(p, g, act, prod, ordered, out, stream);
    // huge strides: a tile's window over several images fits no LDS
    Geometry one = g;
    one.N = 1;
    const Bf16Plan &q = cached_plan(one);
    if (!q.fits) return CPOCONV_ERR_SHAPE;
    for (int n = 0; n < g.N; ++n) {
        const int rc = launch(q, one, act + n * static_cast<int64_t>(g.C) * g.H * g.W, prod, ordered, out + n * static_cast<int64_t>(g.K) * g.Oh * g.Ow, stream);
        if (rc != CPOCONV_OK) return rc;
    }
    return CPOCONV_OK;
}

}  // namespace cpoconv
