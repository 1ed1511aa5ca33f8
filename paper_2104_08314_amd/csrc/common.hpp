// Internal declarations shared by the translation units of libcpoconv.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "cpoconv.h"

namespace cpoconv {

constexpr int kMaxTypes = CPOCONV_MAX_K;   // overlap types 0 .. kw-1
constexpr int kMaxCols = CPOCONV_MAX_I;    // padded columns
constexpr int kLanes = 64;                 // wavefront width on CDNA

// Partition / overlap-type table of a layer (Sections 3.1-3.2), built on the host once per
// call and passed to kernels by value.  "Columns" are the encoded ones (covered by a
// partition and part of the unpadded map) in stream order: overlap type ascending, then
// padded column ascending (which is also first-partition ascending).
struct Geometry {
    int32_t C, H, W, K, kh, kw, stride, pad_h, pad_w;
    int32_t Ih, Iw, Oh, Ow;
    int32_t n_cols;                  // encoded columns
    int32_t n_types;                 // present overlap types
    int32_t nop3;                    // NOP type is the 3-entry segment (no column padding, stride 1)
    int32_t top;                     // overlap type CPS packs, -1 if none
    int32_t top_slot;                // its slot in type_id, -1 if none
    int32_t Kpad;                    // K rounded up to a multiple of 64
    int32_t N;                       // images in the launch (1 unless a batched entry point)
    int32_t channel_last;            // the dense input map is H x W x C instead of C x H x W
    // (whole words: a kernel reads them with scalar loads where the index is the wavefront's, and all of a
    // column with one load where it is the lane's)
    int32_t top_begin, top_end;          // column range of the type CPS packs, empty and past every column if none
    int32_t type_id[kMaxTypes];          // present types, ascending
    int32_t type_begin[kMaxTypes + 1];   // column range of each present type
    uint32_t col[kMaxCols];              // padded column, first partition holding it << 8, column inside that partition << 16
};
__host__ __device__ inline int column_j(const Geometry &g, int i) { return static_cast<int>(g.col[i] & 255u); }
__host__ __device__ inline int column_p0(const Geometry &g, int i) { return static_cast<int>(g.col[i] >> 8 & 255u); }
__host__ __device__ inline int column_what(const Geometry &g, int i) { return static_cast<int>(g.col[i] >> 16); }

// Where element (channel c, row hr, column jr) of one image's dense input map sits.
__device__ __forceinline__ int64_t map_index(const Geometry &g, int c, int hr, int jr)
{
    return g.channel_last ? (static_cast<int64_t>(hr) * g.W + jr) * g.C + c
                          : (static_cast<int64_t>(c) * g.H + hr) * g.W + jr;
}

// An entry of the column table, [image][channel][padded column][band of 64 padded rows]: where the
// column's NZEs of these rows start in DA and which of the rows hold one.  Every padded column has
// its entries; those of a column outside the streams (padding, or under no kernel position) are empty.
struct ColumnEntry {
    int32_t begin;             // absolute offset in DA
    uint32_t rows_lo, rows_hi; // bit r: row 64 * band + r holds an NZE
};

// Does padded column j belong to the streams: part of the unpadded map and under some partition?
__device__ __forceinline__ bool encoded_column(const Geometry &g, int j)
{
    if (j < g.pad_w || j >= g.pad_w + g.W) return false;
    const int first = j < g.kw ? 0 : (j - g.kw + g.stride) / g.stride;   // ceil((j - kw + 1) / stride)
    return first <= min(j / g.stride, g.Ow - 1);
}

// A map the convolution must not read: its encoder gave up (hdr[7] equals the header's stamp), or it holds the other
// algorithm's streams (hdr[3]).  Every kernel on the convolution side leaves its outputs alone then.
__device__ __forceinline__ bool map_unusable(const int32_t *hdr, int image, int algo)
{
    const int32_t *h = hdr + static_cast<int64_t>(image) * 8;
    const int failed_in = h[7];   // stamp of the call in which an encoder unit gave up; hdr[6] >> 8: stamp of the header
    return (failed_in != 0 && failed_in == (h[6] >> 8)) || h[3] != algo;
}

// IN entries: int32, or int16 in a compact map (same values).  The stream pointer is typed int32
// either way; offsets count entries.
__device__ __forceinline__ int load_index(const int32_t *in, int64_t n, int in16)
{
    return in16 ? static_cast<int>(reinterpret_cast<const int16_t *>(in)[n]) : in[n];
}
__device__ __forceinline__ void store_index(int32_t *in, int64_t n, int v, int in16)
{
    if (in16) reinterpret_cast<int16_t *>(in)[n] = static_cast<int16_t>(v);
    else in[n] = v;
}
template <typename P> __device__ __forceinline__ P *index_advance(P *in, int64_t entries, int in16)
{
    using Byte = typename std::conditional<std::is_const<P>::value, const char, char>::type;
    return reinterpret_cast<P *>(reinterpret_cast<Byte *>(in) + entries * (in16 ? 2 : 4));
}

// What a kernel that reads a dense map applies to every value on the way in: the end of the layer
// that produced the map (its bias, then the ReLU that makes the input of Eq. 1 sparse), so the
// activated map itself is never stored.
struct Producer {
    const float *bias;   // one float per channel of the map, or nullptr
    int32_t relu;        // 0: the map is taken as it is (bias unused)
};

// value of a map element of a channel with bias b: z = v + b (one fp32 addition, none without a
// bias), then z if z > 0, else +0.  The test is on the bit pattern (0 < bits <= +inf), so negative
// values, both zeros and NaN give +0 whatever the denormal mode of the comparison would be.
__device__ __forceinline__ float produced(float v, const Producer &prod, float b)
{
    if (prod.relu) {
        if (prod.bias != nullptr) v += b;
        v = (__float_as_uint(v) - 1u) < 0x7f800000u ? v : 0.0f;
    }
    return v;
}

// What a call works out on the host from a layer's shape alone is kept for the next call with that
// shape: per thread, a fixed number of entries (a program has few layers, a slot is overwritten when two
// fall on it).
template <typename Key, typename Value, int kSlots>
class ShapeCache {
public:
    // The value of `key`, made by make(value) if the slot does not hold it; valid until the next call.
    template <typename Make> const Value &get(const Key &key, Make make)
    {
        const int32_t *words = reinterpret_cast<const int32_t *>(&key);
        uint32_t hash = 2166136261u;
        for (size_t i = 0; i < sizeof(Key) / sizeof(int32_t); ++i) hash = (hash ^ static_cast<uint32_t>(words[i])) * 16777619u;
        Slot &slot = slots_[(hash ^ hash >> 15) % kSlots];
        if (!slot.used || memcmp(&slot.key, &key, sizeof(Key)) != 0) {
            slot.used = false;
            make(slot.value);
            slot.key = key;
            slot.used = true;
        }
        return slot.value;
    }

private:
    static_assert(sizeof(Key) % sizeof(int32_t) == 0 && std::is_trivially_copyable<Key>::value, "a key is compared by its words");
    struct Slot {
        bool used = false;
        Key key;
        Value value;
    };
    Slot slots_[kSlots];
};

int check_shape(const cpoconv_shape *s);           // CPOCONV_OK or CPOCONV_ERR_SHAPE
int build_geometry(const cpoconv_shape *s, Geometry *g);
int64_t max_ptr_len(const Geometry &g);
int64_t scratch_bytes_for(const Geometry &g);

void set_hip_error(hipError_t e);

#define CPOCONV_HIP_TRY(expr)                         \
    do {                                              \
        hipError_t e__ = (expr);                      \
        if (e__ != hipSuccess) {                      \
            ::cpoconv::set_hip_error(e__);            \
            return CPOCONV_ERR_HIP;                   \
        }                                             \
    } while (0)

// Measurement aid: while kernel timing is enabled (cpoconv_kernel_timing), every kernel launch is
// bracketed by two HIP events on its own stream.
class KernelTimer {
public:
    KernelTimer(const char *name, hipStream_t stream);
    ~KernelTimer();
    KernelTimer(const KernelTimer &) = delete;
    KernelTimer &operator=(const KernelTimer &) = delete;

private:
    hipStream_t stream_;
    void *stop_;
};

// launchers (defined next to their kernels)
int launch_encode(const float *act, const Producer &prod, const Geometry &g, const cpoconv_map &map, int algo,
                  void *scratch, hipStream_t stream, bool write_columns = false);
int64_t encode_fixed_bytes();                        // look-back words every scratch buffer starts with
int64_t encode_call_flags_bytes(const Geometry &g);  // look-back words of a call that takes two launches
int launch_prepare_weights(const float *w, const Geometry &g, float *wt, hipStream_t stream);
int launch_zero_fill(void *buffer, int64_t bytes, hipStream_t stream);
// convolution over an encoded map (column_table.hip); columns_ready: the encoder of the same call left
// the column table in the scratch buffer
int launch_sparse_conv(const cpoconv_map &map, const Geometry &g, int algo, const float *wt, float *out, void *scratch,
                       hipStream_t stream, bool columns_ready = false);
int64_t column_table_bytes(const Geometry &g);
// 64-row bands of a padded column
__host__ __device__ inline int column_bands(const Geometry &g) { return (g.Ih + kLanes - 1) / kLanes; }
// byte offsets inside the caller's scratch buffer: the encoder's look-back words, then the column table
int64_t scratch_counts_bytes(const Geometry &g);
inline int64_t scratch_columns_offset(const Geometry &g) { return scratch_counts_bytes(g); }
// products on the matrix cores (conv_mfma.hip): over the column table of an encoded map, over a dense map
int launch_conv_columns(const cpoconv_map &map, const ColumnEntry *columns, const Geometry &g, int algo, const float *wt, float *out,
                        hipStream_t stream);
int launch_conv_dense_f32(const float *act, const Producer &prod, const Geometry &g, const float *w, float *out, hipStream_t stream);
int64_t im2col_scratch_bytes(const Geometry &g);
int64_t im2col_weights_bf16_len(const Geometry &g);
int launch_prepare_weights_bf16(const float *w, const Geometry &g, uint16_t *wb, hipStream_t stream);
int launch_im2col_conv(const float *act, const Producer &prod, const Geometry &g, const void *w, void *lowered,
                       float *out, int precision, hipStream_t stream);

}  // namespace cpoconv
