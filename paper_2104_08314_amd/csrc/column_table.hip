// The column table of an encoded map: where the run of NZEs of every (channel, padded column, band of
// 64 padded rows) starts in DA, and which rows of the band hold one.  CPO streams are column-major -
// inside a channel and overlap type the NZEs follow the partitions and, inside a partition's new
// column, the padded rows, ascending - so ptr delimits the runs, and with a bitmap of the rows the
// indices of a run need not be read again: the k-th set bit is the row of the run's k-th NZE.
//
// An encoder that runs in the same call as the convolution leaves the table in the scratch buffer
// (its bitmaps are how it counts); for a map that was encoded in an earlier call it is rebuilt here
// from ptr and IN, a workgroup per (channel, image):
//   1. the channel's ptr entries into LDS (one coalesced read), then per overlap type the absolute DA
//      offset after every partition: Algorithm 2's rule that an entry of -1 stands for the one before
//      it is a running maximum, since live entries are cumulative counts;
//   2. a wavefront per stream column: the partition's NZEs, one lane each, index / kw = padded row,
//      index mod kw = column inside the partition (which holds its columns one after the other);
//   3. a CPS map's overlap-kw type is parsed from the packed stream itself as Algorithm 4 reads it,
//      in parallel: an entry < 0 is a single NZE; a run of entries >= 0 alternates {index of the
//      set's first NZE, pattern}, so an entry's role is the parity of its distance to the last
//      negative entry (a running maximum), the NZE it starts at a running sum, its partition a search
//      over the offsets of step 1, and pattern >> ffs, from the first NZE's row up, the set's rows.
// Nothing is written per NZE.
#include "common.hpp"

#include <algorithm>

namespace cpoconv {

namespace {

constexpr int kTableThreads = 1024;                       // at most; the launch sizes the workgroup to the map
constexpr int kTableWaves = kTableThreads / kLanes;
constexpr int kColumnsAhead = 4;                          // columns whose IN entries a wavefront requests together

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kLanes - 1); }

// inclusive running maximum / sum over the 64 lanes: shifts inside rows of 16 lanes, then the last
// lane of a row to the rows after it
__device__ __forceinline__ int wave_running_max(int v)
{
    constexpr int kLow = static_cast<int>(0x80000000u);   // identity of max
    v = max(v, __builtin_amdgcn_update_dpp(kLow, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLow, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLow, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLow, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLow, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(kLow, v, 0x143, 0xc, 0xf, false));
    return v;
}
__device__ __forceinline__ int wave_running_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// LDS: rows (8 bytes per column and band), run_begin (4 per column), offsets (4 per type and
// partition + 1), entries of ptr (4 each).
__global__ __launch_bounds__(kTableThreads) void column_table_kernel(const Geometry g, const cpoconv_map maps, const int algo,
                                                                    const int bands, ColumnEntry *__restrict__ columns_all)
{
    extern __shared__ unsigned long long table_lds[];
    __shared__ int32_t wave_neg[kTableWaves], wave_out[kTableWaves];
    const int c = blockIdx.x, image = blockIdx.y;
    if (map_unusable(maps.hdr, image, algo)) return;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int nthreads = blockDim.x, nwaves = nthreads / kLanes;
    const int per_type = g.Ow + 1;
    unsigned long long *rows = table_lds;
    int32_t *run_begin = reinterpret_cast<int32_t *>(rows + g.Iw * bands);   // start of a column's run in DA
    int32_t *offsets = run_begin + g.Iw;
    int32_t *segments = offsets + g.n_types * per_type;

    const int in16 = maps.in_bits == 16 ? 1 : 0;
    const int32_t *ptr = maps.ptr + image * maps.ptr_cap;
    const int32_t *indices = index_advance(static_cast<const int32_t *>(maps.in), image * maps.in_cap, in16);
    const int32_t *chan_off = maps.chan_off + static_cast<int64_t>(image) * 3 * (g.C + 1);
    ColumnEntry *out = columns_all + (static_cast<int64_t>(image) * g.C + c) * g.Iw * bands;
    const int cps_top = algo == CPOCONV_ALGO_CPS ? g.top_slot : -1;
    const int seg0 = chan_off[c], seg_len = min(chan_off[c + 1] - seg0, g.n_types * per_type);
    const int da0 = chan_off[(g.C + 1) + c];
    // CPS: the IN entry of a lower-type NZE = the channel's IN offset + the NZE's rank in the channel
    const int in_shift = cps_top >= 0 ? chan_off[2 * (g.C + 1) + c] - da0 : 0;
    const int in_end = cps_top >= 0 ? chan_off[2 * (g.C + 1) + c + 1] : 0;

    for (int i = threadIdx.x; i < seg_len; i += nthreads) segments[i] = ptr[seg0 + i];
    for (int i = threadIdx.x; i < g.Iw * bands; i += nthreads) rows[i] = 0ull;
    for (int i = threadIdx.x; i < g.Iw; i += nthreads) run_begin[i] = 0;
    __syncthreads();
    if (wave == 0) {
        int seg = 0, at = da0;
        const bool npc = segments[0] == CPOCONV_NPC;
        for (int i = 0; i < g.n_types; ++i) {
            int live = 0;   // 0: no NZE, 1: [pType, e_0 .. e_{Ow-1}], 2: the three-entry NOP segment
            if (!npc) live = (g.nop3 && g.type_id[i] == 0) ? 2 : (segments[seg] == CPOCONV_NPF ? 0 : 1);
            int32_t *row = offsets + i * per_type;
            int carry = 0;
            for (int p0 = 0; p0 < g.Ow; p0 += kLanes) {
                const int p = p0 + lane;
                int e = -1;
                if (p < g.Ow) {
                    if (live == 1) e = segments[seg + 1 + p];
                    else if (live == 2) e = p < g.Ow - 1 ? segments[seg + 1] : segments[seg + 2];
                }
                const int m = max(wave_running_max(e), carry);
                if (p < g.Ow) row[1 + p] = at + m;
                carry = __builtin_amdgcn_readlane(m, kLanes - 1);
            }
            if (lane == 0) row[0] = at;
            at += carry;
            seg += npc ? 0 : (live == 2 ? 3 : (live == 1 ? 1 + g.Ow : 1));
        }
    }
    __syncthreads();
    for (int i = 0; i < g.n_types; ++i) {
        const int32_t *row = offsets + i * per_type;
        const int type_end = g.type_begin[i + 1];
        if (i == cps_top) continue;   // packed: below
        for (int v0 = g.type_begin[i] + wave * kColumnsAhead; v0 < type_end; v0 += nwaves * kColumnsAhead) {
            int first[kColumnsAhead];   // the first 64 entries of every column: most columns have no more
#pragma unroll
            for (int u = 0; u < kColumnsAhead; ++u) {
                const int vi = min(v0 + u, type_end - 1), p0 = column_p0(g, vi);
                const int n = row[p0] + lane;
                first[u] = n < row[p0 + 1] ? load_index(indices, n + in_shift, in16) : -1;
            }
#pragma unroll
            for (int u = 0; u < kColumnsAhead; ++u) {
                const int vi = v0 + u;
                if (vi >= type_end) break;
                const int p0 = column_p0(g, vi), j = column_j(g, vi), what = column_what(g, vi);
                const int begin = row[p0], end = row[p0 + 1];   // the partition's NZEs: its columns in turn
                int before = 0;                                 // NZEs of the partition's columns before this one
                for (int n0 = begin; n0 < end; n0 += kLanes) {
                    const int index = n0 == begin ? first[u]
                                                  : (n0 + lane < end ? load_index(indices, n0 + lane + in_shift, in16) : -1);
                    const int h = index / g.kw, column = index - h * g.kw;
                    before += __popcll(__ballot(index >= 0 && column < what));
                    if (index >= 0 && column == what) atomicOr(&rows[j * bands + (h >> 6)], 1ull << (h & 63));
                }
                if (lane == 0) run_begin[j] = begin + before;
            }
        }
    }
    if (cps_top >= 0) {
        const int32_t *bound = offsets + cps_top * per_type;
        const int top_base = bound[0];
        const int e0 = top_base + in_shift;                           // first IN entry of the top type
        const int n_entries = in_end - e0;                            // the top type closes the channel
        int carry_neg = -1;   // position (from e0) of the last negative entry so far
        int carry_out = 0;    // NZEs of the entries so far
        // a lane's entry and the one behind it (the pattern, if the lane's entry leads a pair); the
        // next round's are in flight while this round's are parsed
        auto fetch = [&](int e, int &entry, int &after) {
            entry = e < n_entries ? load_index(indices, e0 + e, in16) : -1;
            after = e + 1 < n_entries ? load_index(indices, e0 + e + 1, in16) : 0;
        };
        int entry_next, after_next;
        fetch(threadIdx.x, entry_next, after_next);
        for (int first = 0; first < n_entries; first += nthreads) {
            const int e = first + threadIdx.x;
            const bool valid = e < n_entries;
            const int entry = entry_next, after = after_next;
            if (first + nthreads < n_entries) fetch(e + nthreads, entry_next, after_next);
            const int m = wave_running_max(entry < 0 ? e : -1);
            if (lane == kLanes - 1) wave_neg[wave] = m;
            __syncthreads();
            int before_neg = carry_neg;
            for (int w = 0; w < wave; ++w) before_neg = max(before_neg, wave_neg[w]);
            const int last_neg = max(m, before_neg);
            const bool leads = valid && entry >= 0 && ((e - last_neg - 1) & 1) == 0;   // the index of a {index, pattern} pair
            const int pattern = leads ? after : 0;
            const int emits = !valid ? 0 : (entry < 0 ? 1 : (leads ? __popc(pattern) : 0));
            const int s = wave_running_sum(emits);
            if (lane == kLanes - 1) wave_out[wave] = s;
            __syncthreads();
            int before_out = carry_out;
            for (int w = 0; w < wave; ++w) before_out += wave_out[w];
            if (emits > 0) {
                const int at = top_base + before_out + s - emits;   // DA position of the entry's first NZE
                int lo = 0, hi = g.Ow - 1;                          // smallest partition whose range ends past it
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (bound[mid + 1] > at) hi = mid; else lo = mid + 1;
                }
                const int index = entry < 0 ? -entry : entry, h = index / g.kw;
                // (the rows of a set lie in one group of four, so never on both sides of a band's edge)
                const unsigned long long set = entry < 0 ? 1ull : static_cast<unsigned long long>(pattern >> (__ffs(pattern) - 1));
                const int j = lo * g.stride + index - h * g.kw;
                atomicOr(&rows[j * bands + (h >> 6)], set << (h & 63));
            }
            int all_neg = carry_neg, all_out = carry_out;
            for (int w = 0; w < nwaves; ++w) { all_neg = max(all_neg, wave_neg[w]); all_out += wave_out[w]; }
            carry_neg = all_neg;
            carry_out = all_out;
            __syncthreads();   // wave_neg / wave_out free for the next round
        }
        // a partition's NZEs: its columns in turn
        for (int vi = g.type_begin[cps_top] + threadIdx.x; vi < g.type_begin[cps_top + 1]; vi += nthreads) {
            int begin = bound[column_p0(g, vi)];
            for (int prev = vi - 1; prev >= g.type_begin[cps_top] && column_p0(g, prev) == column_p0(g, vi); --prev)
                for (int b = 0; b < bands; ++b) begin += __popcll(rows[column_j(g, prev) * bands + b]);
            run_begin[column_j(g, vi)] = begin;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < g.Iw * bands; i += nthreads) {   // columns outside the streams: no run, no rows
        const int j = i / bands;
        int before = 0;
        for (int n = j * bands; n < i; ++n) before += __popcll(rows[n]);
        ColumnEntry entry;
        entry.begin = run_begin[j] + before;
        entry.rows_lo = static_cast<uint32_t>(rows[i]);
        entry.rows_hi = static_cast<uint32_t>(rows[i] >> 32);
        out[i] = entry;
    }
}

}  // namespace

int64_t column_table_bytes(const Geometry &g)
{
    return (static_cast<int64_t>(sizeof(ColumnEntry)) * g.N * g.C * g.Iw * column_bands(g) + 255) / 256 * 256;
}

// Convolution over an encoded map: the column table - left in the scratch buffer by the encoder of the
// same call (columns_ready), rebuilt from the streams otherwise - then the product.
int launch_sparse_conv(const cpoconv_map &map, const Geometry &g, int algo, const float *wt, float *out, void *scratch,
                       hipStream_t stream, bool columns_ready)
{
    ColumnEntry *columns = reinterpret_cast<ColumnEntry *>(static_cast<char *>(scratch) + scratch_columns_offset(g));
    if (!columns_ready) {
        const int bands = column_bands(g);
        const size_t lds = 8 * static_cast<size_t>(g.Iw) * bands + 4 * static_cast<size_t>(g.Iw) +
                           8 * static_cast<size_t>(std::max<int>(g.n_types, 1)) * (g.Ow + 1);
        // a lane per packed entry / four columns per wavefront: one or two rounds of either
        const int threads = std::min(kTableThreads, std::max(256, (g.H * g.W / 2 + kLanes - 1) / kLanes * kLanes));
        KernelTimer timer("column_table", stream);
        hipLaunchKernelGGL(column_table_kernel, dim3(g.C, g.N), dim3(threads), lds, stream, g, map, algo, bands, columns);
        CPOCONV_HIP_TRY(hipGetLastError());
    }
    return launch_conv_columns(map, columns, g, algo, wt, out, stream);
}

}  // namespace cpoconv
