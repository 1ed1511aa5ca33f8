// Convolution on the matrix cores, fp32: the sum over (channel, kernel cell) of Eq. 1 for a tile of
// output positions and kernels, with the input windows expanded in LDS and never in memory.
//
// Two readers fill the windows:
//   columns  the encoded map of Algorithms 1 / 3: the column table says where the run of NZEs of every
//            (channel, padded column, band of 64 padded rows) starts in DA and which rows hold one, so
//            the lane of a window cell finds its NZE (or knows that there is none) from one table
//            entry and two population counts.  IN is not read again, cells without an NZE cost no load.
//   dense    the stored map (the comparator of Section 3.1; lowering happens in LDS addressing), bias
//            and ReLU of a producing layer applied on the way in.
//
// Why the matrix cores for the sparse map too: v_mfma_f32 runs at twice the rate of v_fma_f32 on this
// part and needs no instruction per NZE beyond its expansion.  Walking the NZEs with vector FMAs
// (a scalar bit test, a branch and a broadcast per window cell) reached 20 to 28 TFLOP/s of useful
// sums; at the 40 to 85 % zeros of these maps the product over expanded windows is ahead of that
// everywhere.
//
// Work split: a tile is 16 * MT kernels x 16 * T positions.  A wavefront has a tile of its own, or the
// wavefronts of a workgroup share one: they take the chunks of input channels in turn and their sums are
// added through LDS in wavefront order at the end (results are repeatable).  Per chunk a wavefront fills a
// window of its own (nobody else reads it: no barrier, and while one wavefront waits for its window another
// one multiplies) and multiplies it.  Weights go from memory straight to registers, one to four steps ahead
// - a lane's MT kernels or its four contraction indices are consecutive -, because one operand register
// feeds 32 cycles of matrix work per position tile: LDS could not make them cheaper; the values of the next
// step leave LDS while this one multiplies.
//
// The code is kept short (7 to 14 KB): a launch of one image runs for 5 to 20 us, of which fetching
// instructions is a part; unrolling further or pipelining the windows too made such launches 2 to 5 us
// slower and gained nothing at large batches.
#include "conv_tiles.hpp"

#include <cmath>

namespace cpoconv {

namespace {

constexpr int kStep = 16;              // contraction indices of a step: four matrix instructions of four

struct ConvArgs {
    int32_t C, K, Kpad, N;
    int32_t H, W, pad_h, pad_w;
    int32_t Ih, Iw, Oh, Ow, stride, kw, taps;
    int32_t SW, cols, rows, cells;     // strip width in outputs; window extent behind a tile
    int32_t sets;                      // ceil(cells / 64)
    int32_t cc, nchunks;               // channels of a chunk, chunks
    int32_t tiles, per_m;              // tiles of a strip, of all strips
    int32_t whole_blocks;              // workgroups whose wavefronts have a tile each
    int32_t tab_bytes, window_bytes;   // LDS: offset table, then a window per wavefront
    int32_t bands;                     // 64-row bands of a padded column
    int32_t algo;                      // columns: what hdr[3] has to say
    int32_t relu;
    Divisor by_SW, by_Oh, by_Ih, by_line, by_taps, by_kw, by_tiles, by_per_m;   // line: cols (dense) or rows (columns)
    int64_t map_image, da_image;       // elements between images: dense map, DA
    int32_t map_c, map_r, map_x;       // strides of the dense map
    const float *values;               // the dense map, or DA
    const ColumnEntry *columns;
    const int32_t *hdr;
    const float *bias;
    const float *weights;              // dense: K x C x kh x kw; columns: C x kh x kw x Kpad
    float *out;
};

// One step's weights of a lane: w[mt][j] for kernel kbase + m * MT + mt (m = lane % 16).  Matrix
// instruction j of a step contracts the indices 16 * step + 4 * (lane / 16) + j (a lane's four are
// consecutive).
template <int MT>
struct Weights {
    float w[MT][4];

    // The registers are complete from here on: keeps the compiler from waiting for loads that are issued
    // later when it cannot tell which of several paths filled them.
    __device__ __forceinline__ void settle()
    {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(w[mt][j]));
    }
};

constexpr int kChunk = 16;   // channels of a chunk at most

// wavefronts of a workgroup at most: 128 registers each where a tile's sums fit them
__host__ __device__ constexpr int max_waves(int mt, int t) { return mt * t <= 8 ? 16 : 8; }

template <int MT, int T, bool kDense, bool kFar>
__global__ __launch_bounds__(64 * max_waves(MT, T)) void conv_f32_kernel(const ConvArgs a)
{
    typedef Buffer<kFar> Array;
    typedef typename Array::Offset Offset;
    constexpr int D = MT >= 4 ? 2 : (MT == 2 ? 3 : 5);   // steps whose weights have registers
    extern __shared__ __align__(16) char smem[];
    int32_t *tab = reinterpret_cast<int32_t *>(smem);   // byte offset inside the window of every contraction index of a chunk
    const int lane = lane_id(), n = lane & 15, kk = lane >> 4;
    const int wave = uni(threadIdx.x / kLanes), nwaves = blockDim.x / kLanes;
    char *window = smem + a.tab_bytes + wave * a.window_bytes;
    const int stride_c = a.cells * 4;

    // the last workgroups share a tile: their wavefronts take the chunks in turn
    const bool shared = static_cast<int>(blockIdx.x) >= a.whole_blocks;
    const int first_chunk = shared ? wave : 0, stride_chunk = shared ? nwaves : 1;
    const int number = shared ? a.whole_blocks * nwaves + dealt(blockIdx.x - a.whole_blocks, gridDim.x - a.whole_blocks)
                              : dealt(blockIdx.x, a.whole_blocks) * nwaves + wave;
    const int mb = quotient(number, a.by_per_m), in_m = number - mb * a.per_m;
    const int strip = quotient(in_m, a.by_tiles), tile = in_m - strip * a.tiles;
    const int kbase = mb * 16 * MT, p0 = tile * 16 * T, x0 = strip * a.SW;
    const int row0 = quotient(p0, a.by_SW), in_row0 = p0 - row0 * a.SW;
    const int image0 = quotient(row0, a.by_Oh), y0 = row0 - image0 * a.Oh, top = y0 * a.stride;
    const int positions = a.N * a.Oh * a.SW;

    // weights of the first steps, on their way before anything else
    const Offset Kd = static_cast<Offset>(a.C) * a.taps;
    const Array weights(a.weights, static_cast<int64_t>(Kd) * (kDense ? a.K : a.Kpad) * 4);
    const Offset index_bytes = kDense ? 4u : a.Kpad * 4u;
    constexpr int kAt = kDense ? MT : 4;
    Offset at[kAt];
#pragma unroll
    for (int i = 0; i < kAt; ++i)
        at[i] = kDense ? (static_cast<Offset>(min(kbase + n * MT + i, a.K - 1)) * Kd + 4 * kk) * 4u : ((4 * kk + i) * a.Kpad + min(kbase + n * MT, a.Kpad - MT)) * 4u;
    typedef Weights<MT> W;
    auto load = [&](W &w, uint32_t q) __attribute__((always_inline)) {   // the step of contraction indices q ..
        if constexpr (kDense) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) weights.template load<4>(w.w[mt], at[mt], q * index_bytes);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float f[MT];
                weights.template load<MT>(f, at[j], q * index_bytes);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) w.w[mt][j] = f[mt];
            }
        }
    };
    W w[D];
    const uint32_t q_first = static_cast<uint32_t>(first_chunk) * a.cc * a.taps;
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(w[d], q_first + d * kStep);   // (past a short chunk: not used, past the end: zeros)

    // where the lane's positions start in the window, and in the output (at kernel kbase + 4 * kk * MT; less than
    // nothing: nowhere)
    const int64_t plane = static_cast<int64_t>(a.Oh) * a.Ow;
    int base[T];
    int64_t to[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int p = in_row0 + t * 16 + n, row = quotient(p, a.by_SW), image = quotient(y0 + row, a.by_Oh);
        const int y = y0 + row - image * a.Oh, x = p - row * a.SW;
        const bool exists = p0 + t * 16 + n < positions;
        base[t] = exists ? ((image * a.Ih + y * a.stride - top) * a.cols + x * a.stride) * 4 : 0;
        bool ok = exists && x0 + x < a.Ow;
        if constexpr (!kDense) ok = ok && !map_unusable(a.hdr, min(image0 + image, a.N - 1), a.algo);
        to[t] = ok ? (static_cast<int64_t>(image0 + image) * a.K + kbase + 4 * kk * MT) * plane + y * a.Ow + x0 + x : -1;
    }
    const int chunk_q = a.cc * a.taps;
    auto window_offset = [&](int q) __attribute__((always_inline)) {
        const int c = quotient(q, a.by_taps), tap = q - c * a.taps, l = quotient(tap, a.by_kw);
        return c * stride_c + (l * a.cols + (tap - l * a.kw)) * 4;
    };
    for (int i = threadIdx.x; i < a.tab_bytes / 4; i += blockDim.x) tab[i] = window_offset(min(i, chunk_q - 1));

    const int64_t channel_bytes = kDense ? static_cast<int64_t>(a.map_c) * 4
                                         : static_cast<int64_t>(a.Iw) * a.bands * static_cast<int>(sizeof(ColumnEntry));
    const int64_t image_bytes = kDense ? a.map_image * 4 : a.C * channel_bytes;
    const char *source = (kDense ? reinterpret_cast<const char *>(a.values) : reinterpret_cast<const char *>(a.columns)) + image0 * image_bytes;

    floatx4 acc[MT][T];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < T; ++t) acc[mt][t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- a cell of the window: where it comes from (past the end: no source, reads zero) and goes to, the same
    // for every chunk ------------------------------------------------------------------------------------
    struct Cell {
        Offset from, da;        // columns: da, the cell's image in DA
        int to, row;
        bool inside, ok;
    };
    auto cell_of = [&](int i) __attribute__((always_inline)) {
        Cell cell = {};
        int r, q;
        if constexpr (kDense) { r = quotient(i, a.by_line); q = i - r * a.cols; }
        else { q = quotient(i, a.by_line); r = i - q * a.rows; }
        const int v = top + r, image = quotient(v, a.by_Ih), row = v - image * a.Ih, j = x0 * a.stride + q;
        cell.inside = i < a.cells;
        cell.to = (r * a.cols + q) * 4;
        cell.ok = cell.inside && image0 + image < a.N && j < a.Iw;
        if constexpr (kDense) {
            const int hr = row - a.pad_h, jr = j - a.pad_w;
            cell.ok = cell.ok && hr >= 0 && hr < a.H && jr >= 0 && jr < a.W;
            cell.from = (image * static_cast<Offset>(a.map_image) + static_cast<Offset>(hr) * a.map_r + static_cast<Offset>(jr) * a.map_x) * 4u;
        } else {
            cell.row = row & 63;
            cell.from = ((static_cast<Offset>(image) * a.C * a.Iw + j) * a.bands + (row >> 6)) * sizeof(ColumnEntry);
            cell.da = image * static_cast<Offset>(a.da_image * 4);
            cell.ok = cell.ok && !map_unusable(a.hdr, min(image0 + image, a.N - 1), a.algo);
        }
        cell.from = cell.ok ? cell.from : Array::kNothing;
        return cell;
    };
    const Cell first_cell = cell_of(lane);

#pragma unroll 1
    for (int chunk = first_chunk; chunk < a.nchunks; chunk += stride_chunk) {
        const int c0 = chunk * a.cc, nc = min(a.cc, a.C - c0);
        // ---- the window: lane = cell of 64, all of a chunk's channels on the way together.  Channels past the
        // last one hold anything ---------------------------------------------------------------------------
        const Array buffer(source + c0 * channel_bytes, (a.N - image0) * image_bytes - c0 * channel_bytes);
        Cell cell = first_cell;
#pragma unroll 1
        for (int i = lane;;) {
            float x[kChunk];
            Offset at_channel = 0;
            asm volatile("" : "+s"(at_channel));   // (added up as the loads go: sixteen multiples are not worth their registers)
            if constexpr (kDense) {
#pragma unroll
                for (int c = 0; c < kChunk; ++c, at_channel += static_cast<Offset>(channel_bytes)) x[c] = buffer.load1(cell.from, at_channel);
                if (a.relu) {   // the end of the layer that produced the map; cells outside the map stay zero
#pragma unroll
                    for (int c = 0; c < kChunk; ++c) {
                        if (a.bias != nullptr) x[c] += a.bias[min(c0 + c, a.C - 1)];
                        x[c] = cell.ok && (__float_as_uint(x[c]) - 1u) < 0x7f800000u ? x[c] : 0.0f;
                    }
                }
            } else {
                uint3v e[kChunk];   // ColumnEntry: begin, rows_lo, rows_hi
#pragma unroll
                for (int c = 0; c < kChunk; ++c, at_channel += static_cast<Offset>(channel_bytes)) e[c] = buffer.load3(cell.from, at_channel);
                if (nc < kChunk) {   // channels past the last one: another image's entries, or the end of the table
#pragma unroll
                    for (int c = 0; c < kChunk; ++c) {
                        e[c][1] = c < nc ? e[c][1] : 0u;
                        e[c][2] = c < nc ? e[c][2] : 0u;
                    }
                }
                // the cell's row among the column's rows, and those above it
                const uint32_t bit = 1u << (cell.row & 31), bit_lo = cell.row < 32 ? bit : 0u, bit_hi = cell.row < 32 ? 0u : bit;
                const uint32_t below_lo = cell.row < 32 ? bit - 1u : ~0u, below_hi = cell.row < 32 ? 0u : bit - 1u;
                const Array runs(a.values + image0 * a.da_image, (a.N - image0) * a.da_image * 4);
#pragma unroll
                for (int c = 0; c < kChunk; ++c) {
                    const bool has = ((e[c][1] & bit_lo) | (e[c][2] & bit_hi)) != 0u;
                    const uint32_t where = e[c][0] + __popc(e[c][1] & below_lo) + __popc(e[c][2] & below_hi);
                    x[c] = runs.load1(has ? where * Offset{4} + cell.da : Array::kNothing, 0);
                }
            }
            if (cell.inside) {
                int to_channel = cell.to, cc = a.cc;
                asm volatile("" : "+v"(to_channel), "+s"(cc));
#pragma unroll
                for (int c = 0; c < kChunk; ++c, to_channel += stride_c)
                    if (c < cc) *reinterpret_cast<float *>(window + to_channel) = x[c];
            }
            i += kLanes;
            if (i - lane >= a.sets * kLanes) break;
            cell = cell_of(i);
        }
        if (chunk == first_chunk) __syncthreads();   // the table (every wavefront has a first chunk)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // ---- the product: steps of sixteen contraction indices, the last one masked ------------------------
        const int nq = nc * a.taps, steps = (nq + kStep - 1) / kStep;
        const uint32_t q0 = static_cast<uint32_t>(c0) * a.taps;
        const int4 *offsets = reinterpret_cast<const int4 *>(tab) + kk;
        if (chunk != first_chunk) {
#pragma unroll
            for (int d = 0; d < D - 1; ++d) load(w[d], q0 + d * kStep);
        }
        int4 o = offsets[0];
        float x[D][4][T];   // the values of this step and, on their way, of the next
        auto read = [&](float (&v)[4][T]) __attribute__((always_inline)) {
            const int off[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < T; ++t) v[j][t] = *reinterpret_cast<const float *>(window + (base[t] + off[j]));
        };
        read(x[0]);
        o = offsets[min(1, steps - 1) * 4];
        auto step_of = [&](auto d_, int step) __attribute__((always_inline)) {
            constexpr int d = decltype(d_)::value;
            read(x[(d + 1) % D]);
            o = offsets[min(step + 2, steps - 1) * 4];
            w[d].settle();
            load(w[(d + D - 1) % D], q0 + (step + D - 1) * kStep);
            if (step * kStep + kStep > nq) {   // indices past the chunk's last one: neither weight nor value counts
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool ok = step * kStep + 4 * kk + j < nq;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) w[d].w[mt][j] = ok ? w[d].w[mt][j] : 0.0f;
#pragma unroll
                    for (int t = 0; t < T; ++t) x[d][j][t] = ok ? x[d][j][t] : 0.0f;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[d].w[mt][j], x[d][j][t], acc[mt][t], 0, 0, 0);
        };
#pragma unroll 1
        for (int step = 0; step < steps; step += D) {
            step_of(std::integral_constant<int, 0>(), step);
            if (D > 1 && step + 1 < steps) step_of(std::integral_constant<int, 1 % D>(), step + 1);
            if (D > 2 && step + 2 < steps) step_of(std::integral_constant<int, 2 % D>(), step + 2);
            if (D > 3 && step + 3 < steps) step_of(std::integral_constant<int, 3 % D>(), step + 3);
            if (D > 4 && step + 4 < steps) step_of(std::integral_constant<int, 4 % D>(), step + 4);
        }
    }

    // ---- the wavefronts' sums, added in wavefront order; a register holds kernel row 4 * kk + i of the tile
    // of kernels and position n of the tile of positions -----------------------------------------------
    constexpr int kRegs = MT * T * 4;
    float *red = reinterpret_cast<float *>(smem);
    if (shared) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[(wave * kRegs + (t * MT + mt) * 4 + i) * kLanes + lane] = acc[mt][t][i];
        __syncthreads();
    }
    const int left = a.K - kbase - 4 * kk * MT;   // kernels of the lane that exist
    auto store = [&](int reg, float s) __attribute__((always_inline)) {
        const int t = reg / (4 * MT), k = (reg % 4) * MT + (reg / 4) % MT;
        int64_t at = to[0];
#pragma unroll
        for (int u = 1; u < T; ++u) at = t == u ? to[u] : at;
        if (at >= 0 && k < left) a.out[at + k * plane] = s;
    };
    if (shared) {
        for (int reg = wave; reg < kRegs; reg += nwaves) {
            float s = red[reg * kLanes + lane];
            for (int v = 1; v < nwaves; ++v) s += red[(v * kRegs + reg) * kLanes + lane];
            store(reg, s);
        }
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) store((t * MT + mt) * 4 + i, acc[mt][t][i]);
    }
}

// ---- launch shape ----------------------------------------------------------------------------------

struct ConvPlan {
    int mt, t, sw, cc, waves;
    int whole;  // tiles that a wavefront takes alone (in: whether any may be); the others are shared by a workgroup
    bool far;   // a tile's share of an array spans 4 GiB or more: the kernel with 64-bit addresses
    int rows, cols, tiles, strips, mblocks, tab_bytes, window_bytes, lds;
    double cost;
};

bool evaluate(const Geometry &g, bool dense, ConvPlan *p)
{
    const int taps = g.kh * g.kw, nb = 16 * p->t;
    p->rows = window_rows(g, nb, p->sw);
    p->cols = (p->sw - 1) * g.stride + g.kw;
    const int cells = p->rows * p->cols, sets = (cells + kLanes - 1) / kLanes;
    const int64_t positions = static_cast<int64_t>(g.N) * g.Oh * p->sw;
    if (positions >= (int64_t{1} << 31) - 4096 || cells >= 65535) return false;
    const int64_t images = std::min<int64_t>(g.N, (nb - 1) / (static_cast<int64_t>(g.Oh) * p->sw) + 2), below = (int64_t{1} << 32) - 4096;
    const int64_t chw = static_cast<int64_t>(g.C) * g.H * g.W, entries = static_cast<int64_t>(g.C) * g.Iw * column_bands(g);
    const int64_t weights_bytes = static_cast<int64_t>(g.C) * taps * (dense ? g.K : g.Kpad) * 4;
    p->far = 4 * chw * images >= below || weights_bytes >= below || (!dense && sizeof(ColumnEntry) * entries * images >= below);
    if (p->far && (p->mt > 1 || p->t > 1)) return false;
    p->tiles = static_cast<int>((positions + nb - 1) / nb);
    p->strips = (g.Ow + p->sw - 1) / p->sw;
    p->mblocks = (g.K + 16 * p->mt - 1) / (16 * p->mt);
    const int64_t blocks = static_cast<int64_t>(p->tiles) * p->strips * p->mblocks;
    const int nchunks = (g.C + p->cc - 1) / p->cc;
    const int steps = (p->cc * taps + kStep - 1) / kStep;
    p->tab_bytes = steps * kStep * 4;
    p->window_bytes = (p->cc * cells * 4 + 15) / 16 * 16;
    int waves = std::min(std::min(nchunks, p->waves), max_waves(p->mt, p->t));
    while (waves > 1 && p->tab_bytes + static_cast<int64_t>(waves) * p->window_bytes > kLdsLimit) --waves;
    const int rounds = (nchunks + waves - 1) / waves;
    p->waves = waves = (nchunks + rounds - 1) / rounds;
    p->whole = waves == 1 ? static_cast<int>(std::min<int64_t>(blocks, INT32_MAX)) : (p->whole ? static_cast<int>(blocks / 1024 * 1024 / waves) * waves : 0);
    p->lds = std::max(p->tab_bytes + waves * p->window_bytes, waves > 1 ? waves * p->mt * p->t * 1024 : 0);
    if (p->lds > kLdsLimit || blocks >= (int64_t{1} << 31)) return false;
    // Estimated cycles.  Vector instructions do not overlap with fp32 matrix instructions on this part, so
    // what a wavefront spends per chunk adds up: matrix instructions (32 cycles each), the loads and
    // additions around them, filling its window.  Then the load of the busiest SIMD - whole tiles first, then
    // the shared ones -, the latency of a lone wavefront, and the weights' way out of the L2.  The constants
    // are fitted to 37 layers of 1 to 32 images x every launch shape below, dense and columns, on MI355X: the
    // shape picked is 3 % slower than the best one on average.
    const double step = p->mt * p->t * 128.0 + 6.6 + 47.9 * p->t + 0.9 * p->mt;
    const double chunk = steps * step + sets * p->cc / 16.0 * (dense ? 1720.0 : 1070.0) + 625.0;
    const double store = p->mt * p->t * 175.0;
    const double alone_in_tile = nchunks * chunk + 1500.0 + store, sharing = rounds * chunk + 1500.0 + 3.0 * store;
    double whole = p->whole / 1024.0;   // per SIMD
    if (waves == 1) whole = whole <= 5.0 ? std::ceil(whole) : whole + 0.32;
    const int64_t rest = blocks - p->whole;
    const double per_unit = rest / static_cast<double>(kComputeUnits);
    double shared = (per_unit <= 8.0 ? std::ceil(per_unit) : per_unit + 0.16) * waves / 4.0;
    if (waves < 4 && rest > 0) shared = rest * waves < 4096 ? std::ceil(rest * waves / 1024.0) : (per_unit + 0.16) * waves / 4.0;
    const int resident = std::max(1, std::min(4 * (p->mt * p->t >= 8 ? 4 : 5) / waves, kLdsLimit / p->lds));
    const double active = std::min(resident * waves / 4.0, std::max(whole + shared, 1.0));
    const double through = (whole * alone_in_tile + shared * sharing) * (1.0 + 0.47 / active);
    const double alone = (p->whole > 0 ? nchunks : rounds) * (steps * (step + 582.0) + sets * (dense ? 5840.0 : 3760.0)) + 11300.0;
    const double weights = blocks / static_cast<double>(kComputeUnits) * 16.0 * p->mt * g.C * taps * 4.0 / 146.0 * (dense ? 1.6 : 1.0);
    p->cost = std::max(through, alone) + weights;
    return true;
}

// The launch shape with the smallest estimate.  A tile belongs to a wavefront alone where there are enough of them
// (no additions at the end), rounded down to a multiple of the 1024 SIMDs; the tiles left over - and all
// of them in small launches - are shared by the wavefronts of a workgroup, so that the last round is a short
// one (128@56, 32 images: 285 -> 270 us, 5x5 64@27: 146 -> 131).  Kernels and positions of a wavefront, strips as wide as a
// small map or eight or four columns (compact windows), chunks of sixteen channels (whole steps whatever
// the kernel), fewer for layers of few channels or where a window of sixteen does not fit.
ConvPlan conv_plan(const Geometry &g, bool dense)
{
    ConvPlan best;
    best.cost = -1.0;
    for (int cc : {16, 8, 4, 2, 1}) {
        if (best.cost >= 0.0 && (cc < 4 || (cc < 16 && g.C >= 48) || (cc == 4 && g.C > 24))) continue;
        if (cc > 1 && cc / 2 >= g.C) continue;
        for (int mt : {4, 2, 1}) {
            if (mt > 1 && 8 * mt >= g.K) continue;
            for (int t : {2, 1})
                for (int sw : {g.Ow, 8, 4}) {
                    if (sw > g.Ow || (sw > 20 && g.Ow >= 8)) continue;
                    for (int waves : {1, 2, 4, 8, 16}) {
                        if (waves > 1 && waves / 2 * cc >= g.C) break;
                        for (int whole : {0, 1}) {
                            ConvPlan p;
                            p.mt = mt; p.t = t; p.sw = sw; p.cc = std::min(cc, g.C); p.waves = waves; p.whole = whole;
                            if (evaluate(g, dense, &p) && (best.cost < 0.0 || p.cost < best.cost)) best = p;
                        }
                    }
                }
        }
    }
    if (best.cost < 0.0) {   // large strides: the least window there is
        best.mt = best.t = best.sw = best.cc = best.waves = 1;
        best.whole = 0;
        if (!evaluate(g, dense, &best)) best.cost = -1.0;
    }
    return best;
}

const ConvPlan &cached_plan(const Geometry &g, bool dense)
{
    struct Key {
        int32_t C, H, W, K, kh, kw, stride, pad_h, pad_w, N, channel_last, dense;
    };
    static thread_local ShapeCache<Key, ConvPlan, 128> cache;
    const Key key = {g.C, g.H, g.W, g.K, g.kh, g.kw, g.stride, g.pad_h, g.pad_w, g.N, g.channel_last, dense ? 1 : 0};
    return cache.get(key, [&](ConvPlan &p) { p = conv_plan(g, dense); });
}

template <bool kDense>
int launch(const ConvPlan &p, const ConvArgs &a, const char *name, hipStream_t stream)
{
    KernelTimer timer(name, stream);
    const dim3 grid(p.tiles * p.strips * p.mblocks - p.whole + p.whole / p.waves), block(p.waves * kLanes);
    if (p.far) hipLaunchKernelGGL((conv_f32_kernel<1, 1, kDense, true>), grid, block, p.lds, stream, a);
#define CPOCONV_CASE(MT, T) \
    else if (p.mt == MT && p.t == T) hipLaunchKernelGGL((conv_f32_kernel<MT, T, kDense, false>), grid, block, p.lds, stream, a);
    CPOCONV_CASE(4, 2) CPOCONV_CASE(4, 1) CPOCONV_CASE(2, 2) CPOCONV_CASE(2, 1) CPOCONV_CASE(1, 2) CPOCONV_CASE(1, 1)
#undef CPOCONV_CASE
    CPOCONV_HIP_TRY(hipGetLastError());
    return CPOCONV_OK;
}

ConvArgs make_args(const Geometry &g, const ConvPlan &p, bool dense)
{
    ConvArgs a = {};
    a.C = g.C; a.K = g.K; a.Kpad = g.Kpad; a.N = g.N;
    a.H = g.H; a.W = g.W; a.pad_h = g.pad_h; a.pad_w = g.pad_w;
    a.Ih = g.Ih; a.Iw = g.Iw; a.Oh = g.Oh; a.Ow = g.Ow; a.stride = g.stride; a.kw = g.kw; a.taps = g.kh * g.kw;
    a.SW = p.sw; a.cols = p.cols; a.rows = p.rows; a.cells = p.cols * p.rows;
    a.sets = (a.cells + kLanes - 1) / kLanes;
    a.cc = p.cc; a.nchunks = (g.C + p.cc - 1) / p.cc;
    a.tiles = p.tiles; a.per_m = p.tiles * p.strips;
    a.whole_blocks = p.whole / p.waves;
    a.tab_bytes = p.tab_bytes; a.window_bytes = p.window_bytes;
    a.by_SW = divisor(p.sw); a.by_Oh = divisor(g.Oh); a.by_Ih = divisor(g.Ih); a.by_line = divisor(dense ? p.cols : p.rows);
    a.by_taps = divisor(a.taps); a.by_kw = divisor(g.kw); a.by_tiles = divisor(p.tiles); a.by_per_m = divisor(a.per_m);
    a.bands = column_bands(g);
    return a;
}

// A launch for the whole batch; with huge strides, where the window of a tile over several images may fit no
// LDS, one for every image.  fill(args, n): the arrays, from image n on.
template <bool kDense, typename Fill>
int launch_batch(const Geometry &g, const char *name, hipStream_t stream, const Fill &fill)
{
    auto go = [&](const Geometry &geometry, const ConvPlan &p, int n) {
        ConvArgs a = make_args(geometry, p, kDense);
        fill(a, n);
        return launch<kDense>(p, a, name, stream);
    };
    const ConvPlan &p = cached_plan(g, kDense);
    if (p.cost >= 0.0) return go(g, p, 0);
    Geometry one = g;
    one.N = 1;
    const ConvPlan &q = cached_plan(one, kDense);
    if (q.cost < 0.0) return CPOCONV_ERR_SHAPE;
    for (int n = 0; n < g.N; ++n) {
        const int rc = go(one, q, n);
        if (rc != CPOCONV_OK) return rc;
    }
    return CPOCONV_OK;
}

}  // namespace

int launch_conv_columns(const cpoconv_map &map, const ColumnEntry *columns, const Geometry &g, int algo, const float *wt, float *out,
                        hipStream_t stream)
{
    return launch_batch<false>(g, "spmv_conv", stream, [&](ConvArgs &a, int n) {
        a.algo = algo;
        a.da_image = map.da_cap;
        a.values = map.da + n * map.da_cap;
        a.columns = columns + static_cast<int64_t>(n) * g.C * g.Iw * column_bands(g);
        a.hdr = map.hdr + n * 8;
        a.weights = wt;
        a.out = out + static_cast<int64_t>(n) * g.K * g.Oh * g.Ow;
    });
}

int launch_conv_dense_f32(const float *act, const Producer &prod, const Geometry &g, const float *w, float *out, hipStream_t stream)
{
    return launch_batch<true>(g, "im2col_conv_f32", stream, [&](ConvArgs &a, int n) {
        a.relu = prod.relu;
        a.bias = prod.bias;
        a.map_image = static_cast<int64_t>(g.C) * g.H * g.W;
        a.map_c = g.channel_last ? 1 : g.H * g.W;
        a.map_r = g.channel_last ? g.W * g.C : g.W;
        a.map_x = g.channel_last ? g.C : 1;
        a.values = act + n * a.map_image;
        a.weights = w;
        a.out = out + static_cast<int64_t>(n) * g.K * g.Oh * g.Ow;
    });
}

}  // namespace cpoconv
