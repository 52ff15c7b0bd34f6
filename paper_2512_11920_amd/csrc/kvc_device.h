// Device-side helpers shared by the kernel files: wave64 primitives (DPP), page-task resolution,
// pool reservation and copy-out.
#pragma once
#include "kvc_common.h"

namespace kvc {

// Debug build (-DKVC_DEBUG_BOUNDS=1): every LDS slot index and pool span the kernels compute is checked
// against its bounds; a violation sets status bit 8 instead of being executed silently.  Off by default.
#ifndef KVC_DEBUG_BOUNDS
#define KVC_DEBUG_BOUNDS 0
#endif
#if KVC_DEBUG_BOUNDS
#define KVC_CHECK(st, cond)                        \
    do {                                           \
        if (!(cond)) atomicOr(&(st)->status, 8u);  \
    } while (0)
#else
#define KVC_CHECK(st, cond) \
    do {                    \
    } while (0)
#endif

constexpr int kWavesPerWG = 4;
constexpr int kThreads = kWavesPerWG * 64;

// LDS bytes reserved for one page's payload under construction: header + bodies can reach
// E + E/64 bytes before the INT8 fallback is chosen, plus slack for the 3-dword body writes.
template <int MAXP>
struct Slot {
    static constexpr int kBytes = ((MAXP * 520 + 16 + 15) / 16) * 16;
    static constexpr int kWords = kBytes / 4;
};

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// Lanes of one wave exchange data through LDS: keep the compiler from moving accesses across.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// DPP data movement.  CTRL: 0x00-0xFF quad_perm, 0x110+n row_shr:n, 0x100+n row_shl:n,
// 0x140 row_mirror, 0x141 row_half_mirror, 0x142 row_bcast:15, 0x143 row_bcast:31.
// Lanes whose source is outside the row, or whose row is not in ROW_MASK, receive `old`.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, CTRL, ROW_MASK, 0xF, false);
}

// max over the wave, result uniform (read from lane 63)
__device__ __forceinline__ uint32_t wave_max_dpp(uint32_t v) {
    v = max(v, dpp<0xB1>(0, v));        // quad_perm [1,0,3,2]
    v = max(v, dpp<0x4E>(0, v));        // quad_perm [2,3,0,1]
    v = max(v, dpp<0x141>(0, v));       // row_half_mirror
    v = max(v, dpp<0x140>(0, v));       // row_mirror: every lane holds its row's max
    v = max(v, dpp<0x142, 0xA>(0, v));  // rows 1,3 take lane 15 of the row before
    v = max(v, dpp<0x143, 0xC>(0, v));  // rows 2,3 take lane 31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_incl_scan_dpp(uint32_t v) {
    v += dpp<0x111>(0, v);
    v += dpp<0x112>(0, v);
    v += dpp<0x114>(0, v);
    v += dpp<0x118>(0, v);
    v += dpp<0x142, 0xA>(0, v);
    v += dpp<0x143, 0xC>(0, v);
    return v;
}

// inclusive prefix sum over quads of a value that is uniform within each quad of lanes
__device__ __forceinline__ uint32_t quad_incl_scan_dpp(uint32_t v) {
    v += dpp<0x114>(0, v);
    v += dpp<0x118>(0, v);
    v += dpp<0x142, 0xA>(0, v);
    v += dpp<0x143, 0xC>(0, v);
    return v;
}

// inclusive prefix sum within each row of 16 lanes
__device__ __forceinline__ uint32_t row16_incl_scan_dpp(uint32_t v) {
    v += dpp<0x111>(0, v);
    v += dpp<0x112>(0, v);
    v += dpp<0x114>(0, v);
    v += dpp<0x118>(0, v);
    return v;
}

// ---- bit strings wider than 32 bits, handled as 32-bit halves --------------------------------
// No 64-bit shift by a register amount may appear in these kernels.  What was observed: one build of one
// encoder instantiation (256 channels, run-time scheme, exactly 128 VGPRs) wrote wrong body bytes for a
// few pages in a thousand, differently on every launch, only when two or more workgroups shared a compute
// unit, and every recompile that moved registers made the fault vanish.  That build held the count of a
// v_lshlrev_b64 in the last VGPR of its allocation; the working hypothesis is that v_lshlrev_b64 /
// v_lshrrev_b64 misread a count held there when another wave shares the SIMD.  The cause was not
// established beyond that (a compiler or occupancy-dependent fault in that one build fits the same
// symptoms).  The rule is harmless either way: packing and unpacking below use 32-bit shifts, funnel
// shifts and byte permutes only; a test scans the generated code for 64-bit shifts by a vector register, and
// the guard that matters is the test that runs every kernel instantiation at full occupancy against
// the CPU reference.

// u[0..7], each below 2^c with 0 <= c <= 8, as one little-endian bit string of 8c bits: x = low 32
// bits, y = the rest.  (c = 9, a run packet, gives a value the caller discards.)
__device__ __forceinline__ uint2 pack8_bits(const uint32_t (&u)[8], uint32_t c) {
    const uint32_t a01 = u[0] | (u[1] << c), a23 = u[2] | (u[3] << c);
    const uint32_t a45 = u[4] | (u[5] << c), a67 = u[6] | (u[7] << c);
    const uint32_t c2 = c << 1;
    const uint32_t b0 = a01 | (a23 << c2), b1 = a45 | (a67 << c2);  // 4c bits each
    // b1 << 4c over 64 bits is (b1 : 0) funnel-shifted right by 32 - 4c; 4c = 32 gives (b1 : 0) itself,
    // and 4c = 0 only occurs with b1 = 0.  The funnel shift reads its amount mod 32, so -4c will do.
    const uint32_t r = (uint32_t)__mul24((int)c, -4);
    return make_uint2(b0 | __builtin_amdgcn_alignbit(b1, 0u, r), __builtin_amdgcn_alignbit(0u, b1, r));
}

// The three dwords of (W.y : W.x) << 8k, k = B mod 4: one byte permute each with a common selector
// {7-k, 6-k, 5-k, 4-k}, which is the byte string 08 07 .. 01 shifted right by 3 - k bytes (the byte
// funnel shift reads its amount mod 4, so ~B will do).
__device__ __forceinline__ void shl_bytes(uint2 W, uint32_t B, uint32_t& d0, uint32_t& d1, uint32_t& d2) {
    const uint32_t sel = __builtin_amdgcn_alignbyte(0x08070605u, 0x04030201u, ~B);
    d0 = __builtin_amdgcn_perm(W.x, 0u, sel);
    d1 = __builtin_amdgcn_perm(W.y, W.x, sel);
    d2 = __builtin_amdgcn_perm(0u, W.y, sel);
}

// element offset of a page inside a cache buffer
__device__ __forceinline__ int64_t page_base(const Geometry& g, int64_t blk, int pg) {
    return blk * g.block_stride + (int64_t)pg * g.page_stride;
}

// element offset, relative to the page base, of dense element index e (token e/d, channel e%d); d is
// any multiple of 32, the quotient comes from a multiplication (checked for every e when a context is made)
__device__ __forceinline__ int64_t elem_off(const Geometry& g, int e) {
    const uint32_t row = ((uint32_t)e * g.d_magic) >> 22;
    return (int64_t)row * g.row_stride + ((uint32_t)e - row * (uint32_t)g.d);
}

// Workgroup index used for task assignment.  Workgroups are dealt round-robin to the 8 XCDs; here each XCD gets one
// contiguous eighth of the tasks, so that it streams through a region of its own, in both directions: the payloads of
// eight distant regions then lie side by side in the pool, and the decoder's XCDs read them side by side again.  A
// million pages of 16 x 128, us, with the encoder's tasks dealt in order -> by eighths: encoder 1075 -> 1051, decoder
// 1077 -> 1048 on the pool it leaves.
__device__ __forceinline__ unsigned task_block_index() {
    const unsigned b = blockIdx.x;
    const unsigned q = gridDim.x >> 3;
    return b < (q << 3) ? (b & 7u) * q + (b >> 3) : b;
}

// A value every lane of the wave holds the same copy of, moved to scalar registers: index arithmetic
// on it (64-bit multiplies, bounds checks) then runs on the scalar unit, loads indexed by it become
// scalar loads, and an access at kernel-argument pointer + such an offset needs no per-lane base.
__device__ __forceinline__ int32_t wave_uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Lane i's value in scalar registers.  UNIFORM: every lane holds the same page task.
template <bool UNIFORM>
__device__ __forceinline__ uint32_t of_lane(uint32_t v, int i) {
    return (uint32_t)(UNIFORM ? __builtin_amdgcn_readfirstlane((int)v) : __builtin_amdgcn_readlane((int)v, i));
}
template <bool UNIFORM>
__device__ __forceinline__ uint64_t of_lane(uint64_t v, int i) {
    return (uint64_t)of_lane<UNIFORM>((uint32_t)v, i) | ((uint64_t)of_lane<UNIFORM>((uint32_t)(v >> 32), i) << 32);
}

// Scaling step of Algorithm 2 for a page whose largest magnitude is the finite, non-zero FP16 value
// with bit pattern m: s = amax / 127 and s_inv = 1 / s, each the correctly rounded binary32 quotient,
// without the general division sequence.  amax / 127 is the product with the correctly rounded
// reciprocal of 127, its exact FMA residual and one corrected FMA (Markstein's construction); 1 / s is
// the hardware reciprocal (within 1 ulp) and one Newton step on the FMA residual.  Neither binary32
// range can under- or overflow here (2^-24 <= amax <= 65504).  The domain is the 31,743 FP16
// magnitudes: kvc_page_scales exposes this function so that a test compares every one of them with
// plain IEEE division.
struct PageScale {
    float s, s_inv;
};

__device__ __forceinline__ PageScale page_scale(uint32_t m) {
    const float a = (float)__builtin_bit_cast(_Float16, (unsigned short)m);
    constexpr float kInv127 = 1.0f / 127.0f;
    const float q0 = a * kInv127;
    const float r = __builtin_fmaf(-q0, 127.0f, a);
    PageScale ps;
    ps.s = __builtin_fmaf(r, kInv127, q0);
    const float y0 = __builtin_amdgcn_rcpf(ps.s);
    const float e = __builtin_fmaf(-ps.s, y0, 1.0f);
    ps.s_inv = __builtin_fmaf(e, y0, y0);
    return ps;
}

struct PageResult {
    uint32_t n16;  // payload size in 16-byte units (0 = page skipped)
    uint32_t mode;
    float scale;
};

// Page tasks of the encoder, one per lane: lane i of a wave holds page i of the wave's batch, so that the ids and
// modes of all its pages are fetched by one load each.  (Resolved page by page, a call with block ids waited for every
// id, and with it for the page loads under way.)
struct EncLanes {
    bool ok;      // there is a page to encode
    int32_t sb;   // source block
    uint32_t pg;  // page inside the block
    uint64_t di;  // descriptor index
    int scheme;   // mode requested for the page
};

// lane-wise: page task t of the call (t < 2^31).  max_mode: the highest mode a per-block request may name for this
// page shape (higher values are read as it)
__device__ __forceinline__ EncLanes enc_locate(const EncodeArgs& a, bool live, uint32_t t, int max_mode) {
    EncLanes r;
    const uint32_t blk = fast_div(t, a.by_ppb);
    r.pg = t - blk * (uint32_t)a.g.ppb;
    int32_t sb = (int32_t)blk, pb = (int32_t)blk, scheme = a.scheme;
    if (live && a.src_ids) sb = a.src_ids[blk];
    if (live && a.pool_ids) pb = a.pool_ids[blk];
    if (live && a.block_scheme) scheme = min((int)a.block_scheme[blk], max_mode);
    r.sb = sb;
    r.scheme = scheme;
    const bool wanted = live && sb >= 0 && pb >= 0;
    r.di = (uint64_t)(uint32_t)pb * (uint32_t)a.g.ppb + r.pg;
    r.ok = wanted && sb < a.n_cache_blocks && r.di < a.n_desc;
    if (wanted && !r.ok) atomicOr(&a.st->status, KVC_ST_BAD_INDEX);
    return r;
}

// Page tasks of the decoder, one per lane: lane i of a wave holds what there is to know about page i of the
// wave's batch, so that the ids, the table entries and the descriptors of all its pages are fetched by one
// load each.  (Resolved one page after the other, with wave-uniform values, every descriptor was waited for
// before the next one was asked for: at 1 KB pages a wave of four pages spent 70 % of its cycles in those waits.)
enum DecKind : uint32_t {
    kDecSkip = 0,     // nothing to do
    kDecPayload = 1,  // packed or INT8 payload
    kDecRaw = 2,      // stored uncompressed
    kDecZero = 3,     // bad index or descriptor: the page is zero-filled
};
struct DecLanes {
    uint64_t off;   // byte offset of the payload in the pool
    int32_t db;     // output block
    uint32_t pg;    // page inside the block
    float s;
    uint32_t meta;  // n16 | mode << 16 | DecKind << 24
};

// Where a page task comes from and goes to, before the descriptor is looked at.
struct DecPlace {
    bool live, bad_index;  // live = false: no task (the other fields are meaningless)
    int64_t pb;            // pool block (< 0: nothing stored)
    int32_t db;            // output block (< 0: skip)
    uint32_t pg;           // page inside the block
};

// lane-wise: page task t of the call (t < 2^31)
__device__ __forceinline__ DecPlace dec_locate(const DecodeArgs& a, bool live, uint32_t t) {
    DecPlace r;
    r.live = live;
    r.bad_index = false;
    const uint32_t blk = fast_div(t, a.by_ppb);
    r.pg = t - blk * (uint32_t)a.g.ppb;
    r.db = (int32_t)blk;
    r.pb = -1;
    if (a.block_table) {  // translate (layer, sequence, predicted logical block) -> pool block
        const uint32_t per_layer = (uint32_t)a.n_seq * (uint32_t)a.k;  // blocks of one call fit 31 bits
        const uint32_t layer = fast_div(blk, a.by_per_layer);
        const uint32_t sj = blk - layer * per_layer;
        const uint32_t sq = fast_div(sj, a.by_k);
        if (live) {
            const int32_t lb = a.pred[sj];
            r.bad_index = lb >= a.max_blocks;
            if (lb >= 0 && !r.bad_index) {
                const int32_t e = a.block_table[(int64_t)sq * a.max_blocks + lb];
                r.bad_index = e >= a.pool_blocks_per_layer;
                if (e >= 0) r.pb = (int64_t)layer * a.pool_blocks_per_layer + e;
            }
        }
    } else {
        int32_t pb = (int32_t)blk, db = (int32_t)blk;
        if (live && a.pool_ids) pb = a.pool_ids[blk];
        if (live && a.dst_ids) db = a.dst_ids[blk];
        r.pb = pb;
        r.db = db;
    }
    return r;
}

// ---- outstanding-request window (Algorithm 1, WaitCompletion over at most Omega_max transfers) ----
// A workgroup is one transfer engine: it takes the next entry of the issue queue, decodes that block,
// reports completion and takes the next.  The grid has at most Omega workgroups, so never more than
// Omega blocks are in flight; every workgroup leaves as soon as the queue is exhausted.

// A stamp of the notification array.  It orders nothing behind it and need not: the pages that a stamp speaks of were
// written through to the device's memory (store_out) and waited for by every wave before the counts moved that led to the
// stamp.  (A release in its place writes back the XCD's whole L2: 8 us an engine and report, when 256 engines did it.)
__device__ __forceinline__ void window_stamp(long long* at, long long clock) {
    __hip_atomic_store(at, clock, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// An engine leaves: it reports its `mine` blocks, its layer stamps being in memory by then, and the last one to leave closes
// the window (WaitCompletion returns: NotifyGPU(ready)).  So whoever sees the closing stamp sees every layer's, and its clock,
// read after the last block was counted, is the latest of the call.  (Without the wait the count moved while a stamp
// of this lane was still on its way, and another engine could close the window ahead of it.)
__device__ __forceinline__ void window_leave(const WindowArgs& w, uint32_t mine, uint32_t n_issued) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), the other counters unchanged
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (atomicAdd(&w.hdr->done, mine) + mine == n_issued) window_stamp(&w.notify[w.n_layers + 3], max(wall_clock64(), 1ll));
}

// ---- narrow engines, and wide ones of small blocks: turn by turn

// What an engine holds between two turns: a run of consecutive queue entries.
struct WindowTurn {
    uint32_t first;  // index of the first queue entry
    uint32_t count;  // entries in the run; 0 = the queue is exhausted, the engine leaves
    uint32_t at;     // the entry at work
};

// End of a block of an engine: the waves meet with all their stores of it in memory, and only then is the next block's
// payload asked for -- one block per engine is in flight, which is what bounds the call by Omega.  After the last block
// of the run `turn`: report the run's blocks as complete -- count them, stamp the layers whose last transfer was among
// them -- and take the next run of up to hdr->chunk queue entries (the first run needs no ticket: engine b begins with
// the b-th).  Called by all threads of the
// workgroup; `s_turn` is two words of LDS, `slots` the run's queue entries, parked in LDS by wave 0, `mine` the
// blocks this engine has completed; n_issued and chunk are the header's (read once: they share a line with the ticket).
// The run spaces out the bookkeeping, which the other waves wait for.  It is kept short: the decoder's stores
// under the window write through to the device's memory (store_out), so that waiting for them is all it takes to
// publish a block; with a write-back of the XCD's L2 in its place a turn cost about 8 us (256 engines).  And the
// counters every engine shares serve one atomic every 10 to 20 ns whatever the engines are doing, so a turn spends
// two (ticket, the layer's pending count); the count of completed blocks is added up per engine and reported when
// the engine leaves.
// Thread 0 does the bookkeeping between two barriers, so the single-lane region lies inside the loop
// body and not across its back edge, and the result comes back in scalar registers: the engines' loop
// and its exit branch on the scalar unit and every wave meets every barrier with all of its lanes.  (With
// the single-lane work at both ends of the loop body the compiler merges it across the back edge into
// an outer loop and lets the other lanes run ahead to the next barrier: the workgroup then never
// meets.)
template <bool FIRST>
__device__ __forceinline__ WindowTurn window_next(const WindowArgs& w, uint32_t* s_turn, WindowTurn turn, const int32_t* slots, uint32_t& mine,
                                                  uint32_t n_issued, uint32_t chunk) {
    // every wave's stores have reached memory before the workgroup meets, and the counters move after that
    if (!FIRST) {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), the other counters unchanged
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    }
    __syncthreads();
    if (!FIRST && ++turn.at < turn.count) return turn;
    mine += turn.count;
    if (threadIdx.x == 0) {
        const long long finished = max(wall_clock64(), 1ll);  // read before the blocks are counted
        const unsigned int t = FIRST ? blockIdx.x * chunk : atomicAdd(&w.hdr->ticket, chunk);
        if (!FIRST) {
            uint32_t i = 0;
            while (i < turn.count) {  // the run's entries are in layer order: one decrement per layer met
                const uint32_t l_rel = fast_div((uint32_t)slots[i], w.by_per_layer);
                uint32_t n = 1;
                while (i + n < turn.count && fast_div((uint32_t)slots[i + n], w.by_per_layer) == l_rel) ++n;
                if (atomicSub(&w.pending[l_rel], (int)n) == (int)n)
                    window_stamp(&w.notify[w.layer_begin + (int32_t)l_rel], finished);
                i += n;
            }
            if (t >= n_issued) window_leave(w, mine, n_issued);
        }
        s_turn[0] = t;
        s_turn[1] = t < n_issued ? min(chunk, n_issued - t) : 0u;
    }
    __syncthreads();
    WindowTurn r;
    r.first = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_turn[0]);
    r.count = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_turn[1]);
    r.at = 0;
    return r;
}

// ---- the other wide engines: looked ahead for

constexpr uint32_t kWindowNone = ~0u;

// The kernel's arguments, read from where the launch put them (a kernel of one argument).  What only a rare part of a
// kernel needs is asked for there and not held in scalar registers meanwhile (an engine has some 80 words of arguments and
// 30 of books, and 100 scalar registers).
template <class T>
__device__ __forceinline__ const T& params_again() {
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const T*)(const void*)p;
}

// What the clerk of a wide engine knows (wave-uniform): the entries ahead of the engine, and the blocks behind it.
// Entries come in runs, `left` of them from `next` on, `step` apart, a run asked for before the last entry of the run before
// is used up.  The first run needs no ticket: entries in a row where the call's runs are that long anyway, else kWindowAhead
// entries that lie `engines` apart: in a row, the first layers would wait for a few engines' fourth block while the others are
// at work on later ones.  (256 engines, first layer ready and whole call, us, in a row / apart: 2,560 blocks of 32 pages of 16 x 256
// in ten layers 71 and 142.7 / 32 and 138.8; 2,048 of eight in eight layers 23.5 and 44.5 / 12.8 and 45.5.)
struct WindowBooks {
    uint32_t n_issued, engines;
    uint32_t next, left, step, size;
    uint32_t open;            // the queue may hold more than the known run
    int32_t slot1, slot2;     // slots of the two blocks after the one at work (-1: none),
    int32_t pb1;              // and the pool block of the first
    uint32_t mine;            // blocks completed,
    uint32_t acc, layer;      // those of them not yet reported, all of this layer,
    uint32_t rep, rep_layer;  // and those to report

    __device__ __forceinline__ void get(const WindowBooks& from) {
        constexpr int n = sizeof(WindowBooks) / 4;
        uint32_t v[n];
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = (uint32_t)wave_uniform((int32_t)reinterpret_cast<const uint32_t*>(&from)[i]);
        *this = __builtin_bit_cast(WindowBooks, v);
    }
    __device__ __forceinline__ void put(WindowBooks& to) const {
        wave_sync();
        if (lane_id() == 0) to = *this;
        wave_sync();
    }

    __device__ __forceinline__ void open_at(uint32_t issued, uint32_t engine, uint32_t n_engines, uint32_t chunk) {
        const bool rows = chunk >= (uint32_t)kWindowAhead;
        n_issued = issued;
        engines = n_engines;
        left = max(chunk, (uint32_t)kWindowAhead);
        next = rows ? engine * left : engine;
        step = rows ? 1u : n_engines;
        size = chunk;
        open = 1;
        mine = acc = rep = rep_layer = 0;
    }
    __device__ __forceinline__ uint32_t take() {
        if (left == 0) return kWindowNone;
        const uint32_t i = next;
        next += step;
        --left;
        return i < n_issued ? i : kWindowNone;
    }
    // Length of the run to ask for now (0: none): the call's chunk, halved when less than two such runs per engine seem to
    // be left, so that the engines end within a block of each other.  (Every run is an atomic on one counter, which
    // serves one every 10 to 20 ns whoever asks: a few hundred engines can ask for every block.)
    __device__ __forceinline__ uint32_t next_run() {
        if (left != 0 || open == 0) return 0u;
        const uint32_t rest = next < n_issued ? n_issued - next : 0u;
        while (size > 1 && rest < 2u * engines * size) size >>= 1;
        return size;
    }
    __device__ __forceinline__ void refill(uint32_t ticket, uint32_t run) {
        open = ticket < n_issued ? 1u : 0u;
        next = ticket;
        left = open ? min(run, n_issued - ticket) : 0u;
        step = 1;
    }
    static __device__ __forceinline__ uint32_t layer_of(const WindowArgs& w, int32_t s) { return s < 0 ? kWindowNone : fast_div((uint32_t)s, w.by_per_layer); }
    // the block at work is decoded: consecutive blocks of a layer are reported together
    __device__ __forceinline__ void block_done(const WindowArgs& w) {
        const uint32_t layer1 = layer_of(w, slot1);
        ++mine;
        ++acc;
        rep = 0;
        if (layer1 != layer || acc >= (uint32_t)kMaxWindowTurn) {
            rep = acc;
            rep_layer = layer;
            acc = 0;
            layer = layer1;
        }
    }
};

// The codec kernels are specialised at compile time for the page shape (kvc_codec.h): d channels, np
// passes of 512 elements, and whether the page fills its last pass (exact: d * N = 512 * np) or not
// (partial: the token count N is read at run time).  These are the host-side entry points of one shape.
// The shapes are compiled in groups (kvc_codec.hip), one lookup function per group; shape_kernels() finds
// the set for N tokens x d channels (nullptr: N * d exceeds eight passes).
struct ShapeKernels {
    int d, np;
    bool partial;
    hipError_t (*compress)(const EncodeArgs& a, hipStream_t s);
    hipError_t (*decompress)(const DecodeArgs& a, hipStream_t s);
    hipError_t (*decompress_window)(const DecodeArgs& a, const WindowArgs& w, unsigned grid, bool wide, hipStream_t s);
    int (*window_capacity)(bool wide, int ppb);  // window engines resident on the current device at once (0: unknown)
    bool (*window_looks_ahead)(int ppb);         // whether the wide ones look ahead
};
constexpr int kShapeGroups = 16;
using ShapeLookup = const ShapeKernels* (*)(int d, int np, bool partial);
#define KVC_DECLARE_GROUP(G) const ShapeKernels* shape_kernels_group##G(int d, int np, bool partial);
KVC_DECLARE_GROUP(0) KVC_DECLARE_GROUP(1) KVC_DECLARE_GROUP(2) KVC_DECLARE_GROUP(3) KVC_DECLARE_GROUP(4) KVC_DECLARE_GROUP(5)
KVC_DECLARE_GROUP(6) KVC_DECLARE_GROUP(7) KVC_DECLARE_GROUP(8) KVC_DECLARE_GROUP(9) KVC_DECLARE_GROUP(10) KVC_DECLARE_GROUP(11)
KVC_DECLARE_GROUP(12) KVC_DECLARE_GROUP(13) KVC_DECLARE_GROUP(14) KVC_DECLARE_GROUP(15)
#undef KVC_DECLARE_GROUP
const ShapeKernels* shape_kernels(int N, int d);

}  // namespace kvc
