// Shared declarations between the C-ABI host code (kvc_api.hip) and the kernels (kvc_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kvc.h"
#include "kvc_fastdiv.h"

namespace kvc {

// Device state block owned by a context.
struct DevState {
    unsigned long long cursor16;  // next free 16-byte unit of the pool
    unsigned int status;          // sticky KVC_ST_* bits
    unsigned int pad;
    unsigned long long stats[8];  // scratch of kvc_stats: pages[0..5], invalid, payload16
};

// Page geometry and cache layout.  Element (token j, channel i) of page pg of block b sits at
// b*block_stride + pg*page_stride + j*row_stride + i of the cache buffer (all in FP16 elements).
struct Geometry {
    int32_t N, d, ppb, E;  // E = N*d elements per page
    int32_t lpr;           // lanes per token row: d / 8 (a lane owns 8 channels)
    uint32_t d_magic;      // ceil(2^22 / d):   e / d   == (e * d_magic) >> 22   for e < 8192
    int64_t row_stride, page_stride, block_stride;
};

struct EncodeArgs {
    const uint16_t* cache;
    int64_t n_cache_blocks;
    const int32_t* src_ids;
    const int32_t* pool_ids;
    int64_t n_pages;  // n blocks * ppb
    Geometry g;
    int32_t scheme;
    const uint8_t* block_scheme;  // optional: requested mode per block (overrides scheme)
    FastDiv by_ppb;
    uint8_t* pool;
    uint64_t pool_units;  // pool size in 16-byte units
    uint64_t kept_units;  // payloads below this unit of the pool are stored to stay in the last-level cache (see kPoolKeptBytes)
    kvc_desc* desc;
    uint64_t n_desc;
    DevState* st;
};

struct DecodeArgs {
    uint16_t* out;
    int64_t n_out_blocks;
    const int32_t* pool_ids;
    const int32_t* dst_ids;
    int64_t n_pages;
    Geometry g;
    const uint8_t* pool;
    uint64_t pool_units;
    const kvc_desc* desc;
    uint64_t n_desc;
    DevState* st;
    uint64_t near_bytes;  // where the range's first payload lies below this byte of the pool, those from it on are read past the last-level cache (see kDecStreamFrom)
    // gather form (block_table != nullptr): page task t = ((l*n_seq + s)*k + j)*ppb + pg
    const int32_t* block_table;
    const int32_t* pred;
    int32_t max_blocks, n_seq, k, n_layers;
    int64_t pool_blocks_per_layer;
    // divisions of the task resolution: by ppb, and in the gather form by n_seq * k and by k
    FastDiv by_ppb, by_per_layer, by_k;
};

// The last-level cache (256 MB, memory side) keeps what is stored without a streaming hint.  Payloads that go to the
// beginning of a pool are stored so, and a call that brings the blocks back finds them there: compress and decompress of
// one set of blocks, us, with every payload stored past the cache -> so: 65,536 pages of 16 x 128 138 -> 127, half a million
// of 16 x 32 280 -> 253, of 16 x 64 517 -> 503, 98,304 of 24 x 96 226 -> 212; sixteen calls of 65,536 pages, each followed by
// its decode, 2,240 -> 2,216.  Only the beginning, because payloads that push others out of the cache reach the memory in no
// order: with no limit half a million pages of 16 x 128, mode 5, are encoded in 512 us (484 with the hint), and fetched back
// no sooner.  Limits of 128, 192, 208, 224 and 256 MB: 16 x 64 510, 502, 502, 500, 520; 65,536 pages of 16 x 256, a mode per
// block, 274, 268, 268, 271, 282 (278 with the hint).
// What it takes to gain: the blocks come back before much else is stored or read, and the pool is young or was reset.  So the payloads
// that contexts keep, and have not fetched, are that many bytes in all; others' are stored past the cache, or they would push
// each other out.  Sixteen pools of 256 MiB of 16 x 128, all offloaded, then all fetched, us a pool, none kept / each pool's
// beginning / what fits: 141.3 / 144.1 / 139.9, 32 of 64 MiB 44.2 / 46.4 / 43.6 (offload 22.3 / 24.2 / 22.5), 64 of 16 MiB 18.6 / 19.0 / 18.2
// (11.2 / 12.3 / 11.7); each fetched right after its offload 142.4 / 130.9 / 130.7, 44.8 / 41.8 / 41.7, 18.7 / 18.5 / 18.6.  16 x 32, 16 x 64, 16 x 256
// and mode 5 the same.  What it costs others: two reads of 224 MB that the cache would hold, after a compress of 256 MiB, take with
// it 151 -> 158, of 160 MB 134 -> 135, of 96 MB 117 -> 113.
constexpr uint64_t kPoolKeptBytes = 208ull << 20;
// Calls of fewer pages are not kept: it costs the encoder 0.1 to 0.2 us and gives as much to a decoder that follows.  Reset and compress, and decompress
// after it, us, none kept / kept, 16 x 128, mode 1: 8 pages 4.8, 7.0 / 5.0, 7.2, 64 4.9, 7.6 / 5.1, 7.6, 128 4.9, 8.0 / 5.1, 7.85, 512 6.1, 9.7 / 6.2, 9.1.
constexpr int64_t kKeptFromPages = 128;
// Calls that decode a whole range of more payload than the cache holds read what lies beyond that beginning with the
// hint: read plainly, it pushes out the beginning, and then itself, before either is read again.  By the size of the
// pages, as the payloads' (a half to a third of it) is not known here; and only where the range's first payload lies in
// the beginning, which the kernel looks up: a range beyond it has nothing there to protect, and lines that two payloads share
// would be read twice.  16 x 128, mode 3, us, read plainly / with the hint: decode repeated; compress and decompress; decode
// after 2 GB of other traffic; decode repeated of a range that begins 256 MB into the pool (in the last, the hint is not taken):
//   512 MiB   109 / 110      239 / 239      154 / 152      109 / 128
//   576 MiB   134 / 126      269 / 269      177 / 171      136 / 146
//   640 MiB   155 / 141      300 / 299      191 / 185      158 / 160
//     1 GiB   254 / 242      502 / 489      287 / 279      255 / 258
//     2 GiB   510 / 495      994 / 981      542 / 541      512 / 519
//     4 GiB 1,015 / 1,002  1,972 / 1,964  1,044 / 1,050  1,014 / 1,031
//   4.5 GiB 1,144 / 1,132  2,228 / 2,214  1,179 / 1,179  1,138 / 1,158
//     5 GiB 1,272 / 1,255  2,473 / 2,460  1,298 / 1,313  1,273 / 1,290
// The other shapes turn at much the same sizes.  16 x 32, 16 x 64, 24 x 96, 16 x 256 and mode 5 of 16 x 128 win 6 to 12 % of a
// repeated decode at 640 MiB; at 576 16 x 256 loses 3 % and mode 5 2 %.  At 4 GiB they win 0 to 3 % and lose less than 1 % after other
// traffic; at 4.5 GiB 16 x 32, 16 x 256 and mode 5 win nothing and lose 1 % after other traffic.  Raw pages win 2 to 10 % at every size.
constexpr uint64_t kDecStreamFrom = 608ull << 20, kDecStreamTo = 4352ull << 20;

constexpr int kMaxPrefetchK = 32;  // predictions per sequence the slot-reuse policy can plan

// Arguments of the prefetch planner (Algorithm 1: translate, residency filter, slot assignment).
struct PlanArgs {
    const int32_t* block_table;  // [n_seq][max_blocks]
    const int32_t* pred;         // [n_seq][k]
    const int32_t* l1_first;     // [n_seq] or null: logical blocks >= l1_first[s] are GPU-local (L1)
    int32_t max_blocks, n_seq, k, layer_begin, layer_end, n_layers, fill_half;
    int32_t policy;              // 0: slot j for prediction j; 1: keep wanted blocks, fill unwanted slots
    int64_t pool_blocks_per_layer;
    FastDiv by_n_seq;
    int32_t* tags;   // [2][n_layers*n_seq*k]
    int32_t* fetch;  // [n_layers*n_seq*k]
    int32_t* loc;    // [n_layers*n_seq*k]
    DevState* st;
};

// Outstanding-request window of the prefetch path (Algorithm 1: WaitCompletion over at most Omega_max
// concurrent transfers).  The workspace of one call: this header, then one pending counter per layer of
// the call, then the queue of issued transfers (slot indices relative to the call's first slot).
struct WindowHdr {
    unsigned int n_issued;  // entries in the queue (constant while the engines run)
    unsigned int engines;   // transfer engines of the call = min(omega, n_issued): the bound on blocks in flight
    unsigned int chunk;     // queue entries an engine takes per turn (1..kMaxWindowTurn)
    unsigned int pad0[13];
    unsigned int ticket;    // next queue entry to hand out; the two hot counters sit in cache lines of their own
    unsigned int pad1[15];
    unsigned int done;      // blocks completed
    unsigned int pad2[31];
};
static_assert(sizeof(WindowHdr) == 256, "window header is 256 bytes");

constexpr int kMaxWindowTurn = 8;  // queue entries an engine takes in a row, and reports at once, at most
constexpr int kWindowManyEngines = 256;  // more engines than this are used only as far as each has eight transfers
constexpr int kWindowAhead = 4;         // queue entries an engine that looks ahead knows without asking, at least

struct WindowArgs {
    WindowHdr* hdr;
    int32_t* pending;      // [layers of the call]: issued transfers of the layer not yet completed
    int32_t* queue;        // [n_now]
    const int32_t* fetch;  // the call's part of the fetch list: [n_now], pool block or -1
    int32_t n_now;         // slots of the call = layers of the call * per_layer
    int32_t per_layer;     // n_seq * k
    FastDiv by_per_layer;
    int32_t layer_begin, n_layers_call, n_layers;
    int32_t omega;         // engines the decode launch starts at most
    int32_t wide;          // they are of the wide kind
    int32_t ahead;         // queue entries that each of them knows without asking, at least
    long long* notify;     // [n_layers + 4], see kvc.h
};

struct WindowParams {
    DecodeArgs a;
    WindowArgs w;
};

inline uint64_t window_workspace_bytes(int64_t n_blocks, int64_t n_layers_call) {
    return sizeof(WindowHdr) + (uint64_t)((n_layers_call * 4 + 255) / 256 * 256) + (uint64_t)n_blocks * 4;
}

// Launch `kernel` and return the status of this launch itself.  (A launch through the <<<>>> form
// reports failure only through the thread's last-error slot, which may still hold an error left by
// an earlier, unrelated call of the application.)
template <typename T>
struct SameType {
    using type = T;
};
// lds: bytes of LDS per workgroup beside the kernel's own.
template <typename... P>
inline hipError_t launch_kernel_lds(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t s, typename SameType<P>::type... args) {
    void* ptrs[] = {static_cast<void*>(&args)...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, s);
}
template <typename... P>
inline hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t s, typename SameType<P>::type... args) {
    return launch_kernel_lds(kernel, grid, block, 0, s, args...);
}

hipError_t launch_prefetch_plan(const PlanArgs& a, hipStream_t s);
hipError_t launch_window_plan(const PlanArgs& a, const WindowArgs& w, hipStream_t s);
hipError_t launch_decompress_window(const DecodeArgs& a, const WindowArgs& w, hipStream_t s);
int window_engine_capacity(const Geometry& g, bool wide);
bool window_looks_ahead(const Geometry& g);  // whether the wide engines look ahead, or go turn by turn
hipError_t launch_fill_i32(int32_t* p, int32_t v, uint64_t n, hipStream_t s);
hipError_t launch_compress(const EncodeArgs& a, hipStream_t s);
hipError_t launch_decompress(const DecodeArgs& a, hipStream_t s);
hipError_t launch_reset(DevState* st, kvc_desc* desc, uint64_t n_desc, hipStream_t s);
hipError_t launch_set_cursor(DevState* st, uint64_t cursor16, hipStream_t s);
hipError_t launch_stats(DevState* st, const kvc_desc* desc, uint64_t n_desc, hipStream_t s);
hipError_t launch_page_scales(const uint16_t* amax, float* s, float* s_inv, uint64_t n, hipStream_t st);
hipError_t launch_copy(void* dst, const void* src, uint64_t n16, hipStream_t s);

}  // namespace kvc
