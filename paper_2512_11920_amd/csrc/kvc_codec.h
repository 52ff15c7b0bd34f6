// The codec kernels, specialised at compile time for the page shape: D channels (any multiple of 32 up to
// 256) and NP = 1..8 passes of 512 elements.  Two kinds of shape: pages that are a whole number of passes
// (N = NP * 512 / D tokens; 16 x 128 FP16, D = 128 and NP = 4, is the paper's 4 KB page and the shape the
// tuning was done on), where every quantity is a constant and no lane is ever inactive, and -- PARTIAL --
// pages of any other token count that needs NP passes, where the element count is read at run time and the
// last pass is short.  This file holds the templates; kvc_codec.hip instantiates them.
//
// Lane mapping: one wave per page, passes of 512 elements, a lane owns 8 consecutive channels (one 128-bit
// access), a packet group is a quad of lanes, a token row is D/8 neighbouring lanes (one 16-lane DPP row at
// D = 128).  Every cross-lane step is a DPP operation, the per-group statistics (max, width, run test) and
// the offset scans are done on quads.  When D does not divide 512 (96, 160, 192, 224) a token row may begin
// in one pass and end in the next: the delta step and its inverse then carry one value from pass to pass.
// Written plainly the codec is bound by vector-ALU issue long before HBM bandwidth; the instruction count
// per element is kept low enough here that the memory system is the limit.
//
// Encode: Algorithm 2 of the paper (scaling, quantize, delta, run-length encode).
// Decode: Section 3.5.3 (undo run-length coding, prefix sum, dequantize; bypass for raw pages).
#pragma once
#include <type_traits>

#include "kvc_device.h"

namespace kvc {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

// Non-temporal hints for the encoder's streams (its input, and the payloads it stores): measured 4-7 % faster.  (The
// decoder's stores have their own, see store_out.)

// 128-bit global accesses of streamed data (each byte is touched once)
__device__ __forceinline__ uint4 load_stream(const uint4* p) {
    const uint4v v = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream(uint4* p, const uint4& v) {
    uint4v w;
    w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    __builtin_nontemporal_store(w, reinterpret_cast<uint4v*>(p));
}

// Compile-time shape of a page of NP passes with D channels per token.  PARTIAL: the page has fewer
// than NP * 512 elements (more than (NP - 1) * 512); kE, kN, kGroups and kHdr are then upper bounds and
// the run-time values come from page_extent().
template <int D, int NP, bool PARTIAL = false>
struct Page {
    static_assert(D % 32 == 0 && D >= 32 && D <= 256 && NP >= 1 && NP <= 8 && (PARTIAL || (NP * 512) % D == 0), "page shape");
    static constexpr int kD = D;
    static constexpr bool kPartial = PARTIAL;
    static constexpr int kE = NP * 512;       // elements
    static constexpr int kN = kE / D;         // tokens
    static constexpr int kPasses = NP;        // passes of 512 elements
    static constexpr int kGroups = NP * 16;   // packet groups of 32
    static constexpr int kHdr = NP * 8;       // header bytes, 4 bits per group
    static constexpr int kLpr = D / 8;        // lanes per token row
    static constexpr bool kAligned = 512 % D == 0;  // a token row never continues into the next pass
    static constexpr int kRowsPerPass = 512 / D;    // (whole rows; exact when kAligned)
    static constexpr int kRounds = (NP + 1) / 2;    // rounds of 64 lanes x 16 bytes that cover a payload (< kE bytes)
    static constexpr bool kChan = !PARTIAL && kN == 16 && (D == 64 || D == 128 || D == 256);  // mode 5 is built for these pages
};

// Extent of a page: elements, header bytes (4 bits per group of 32, rounded up to a byte) and the number
// of lanes that hold data in the last pass.  Constants unless P::kPartial.  A token row is a multiple of
// four lanes, so a packet group (a quad) and a row are either all data or all beyond the page.
struct Extent {
    uint32_t E, hdr, last;
};
template <class P>
__device__ __forceinline__ Extent page_extent(const Geometry& g) {
    Extent x;
    if (P::kPartial) {
        x.E = (uint32_t)g.E;
        x.hdr = (((uint32_t)g.E >> 5) + 1u) >> 1;
        x.last = ((uint32_t)g.E >> 3) - (uint32_t)(P::kPasses - 1) * 64u;
    } else {
        x.E = P::kE;
        x.hdr = P::kHdr;
        x.last = 64u;
    }
    return x;
}
// does this lane hold data in pass p (p a constant after unrolling: true at compile time except in the
// last pass of a partial page)
template <class P>
__device__ __forceinline__ bool lane_live(const Extent& x, int p) {
    return !P::kPartial || p < P::kPasses - 1 || (uint32_t)lane_id() < x.last;
}

// Where a lane sits in pass 0: token row and position inside the row, both in lanes of 8 channels, and
// the byte offset of its 16 bytes inside the page (row-major deal, and the deal of mode 5).
struct LanePos {
    uint32_t row0, col0, off0, off0_chan;
};
template <class P>
__device__ __forceinline__ LanePos lane_pos(const Geometry& g) {
    const uint32_t lane = (uint32_t)lane_id();
    LanePos lp;
    lp.row0 = lane / P::kLpr;
    lp.col0 = lane % P::kLpr;
    lp.off0 = (lp.row0 * (uint32_t)g.row_stride + lp.col0 * 8u) * 2u;
    lp.off0_chan = P::kD == 64 ? (((lane >> 5) * 8u + (lane & 3u)) * (uint32_t)g.row_stride + ((lane >> 2) & 7u) * 8u) * 2u
                               : ((lane & 3u) * (uint32_t)g.row_stride + (lane >> 2) * 8u) * 2u;
    return lp;
}
// ... and in pass p (p is a constant after unrolling): 64 * p lanes further on.
template <class P>
__device__ __forceinline__ uint32_t pass_col(const LanePos& lp, int p) {
    const uint32_t c = lp.col0 + (uint32_t)((p * 64) % P::kLpr);
    return (!P::kAligned && c >= (uint32_t)P::kLpr) ? c - P::kLpr : c;
}
template <class P>
__device__ __forceinline__ uint32_t pass_row(const LanePos& lp, int p) {
    const uint32_t wrap = (!P::kAligned && lp.col0 + (uint32_t)((p * 64) % P::kLpr) >= (uint32_t)P::kLpr) ? 1u : 0u;
    return lp.row0 + (uint32_t)((p * 64) / P::kLpr) + wrap;
}

// Values of the encoder's SCHEME parameter below zero: the mode is read per page at run time, from modes
// 0..4, or from 0..5 (only built for the page shapes that have mode 5).
constexpr int kSchemeRowMajor = -1;
constexpr int kSchemeAny = -2;

constexpr float kMagic = 12582912.0f;  // 1.5 * 2^23: adding it rounds to an integer, ties to even
constexpr uint32_t kMagicBits = 0x4B400000u;

// max(m, |x|) on two FP16 values, NaN if either is one (as the packed max3 of m, x and -x: one instruction)
__device__ __forceinline__ half2v max_magnitude(half2v m, uint32_t bits) {
    const half2v x = __builtin_bit_cast(half2v, bits);
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, x), -x);
}

// Quantize step on 8 FP16 values: bits of (x * s_inv + M_k), M_k = 1.5*2^23 + 256*k.  The fused
// multiply-add rounds the exact product once, to an integer, ties to even; the low byte of the result
// is q (two's complement).  The per-element bias 256*k makes every difference of neighbouring results
// positive: bits(t_k) - bits(t_{k-1}) = q_k - q_{k-1} + 256.
__device__ __forceinline__ void quantize8_bits(const uint4& raw, float s_inv, uint32_t t[8]) {
    const half8 h = __builtin_bit_cast(half8, raw);
#pragma unroll
    for (int k = 0; k < 8; ++k) t[k] = __float_as_uint(__builtin_fmaf((float)h[k], s_inv, kMagic + 256.0f * (float)k));
}

// Two ways of dealing a page's 128-bit pieces (one token, eight channels = one octet) to the lanes.
// Row-major (CHAN = false): piece number p*64 + lane in pass p.  Channel-pair mode 5 (CHAN = true):
// at D = 128 or 256 lane 4*l + r takes, in pass p, token 4*(p mod 4) + r of octet 16*(p div 4) + l, so
// that the four lanes of a quad hold the 16 tokens of one octet over four passes; at D = 64 (eight octets,
// two passes) lane 32*h + 4*l + r takes token 8*h + 4*p + r of octet l, so that a quad and its partner 32
// lanes away hold the 16 tokens of one octet between them.
template <class P, bool CHAN>
__device__ __forceinline__ int piece_index(int p, int lane) {  // position in row-major piece order
    if (!CHAN) return p * 64 + lane;
    if (P::kD == 64) return (8 * (lane >> 5) + 4 * p + (lane & 3)) * P::kLpr + ((lane >> 2) & 7);
    return (4 * (p & 3) + (lane & 3)) * P::kLpr + 16 * (p >> 2) + (lane >> 2);
}

// plain INT8 payload: codes as bytes, row-major
template <class P, bool CHAN>
__device__ __forceinline__ void store_codes(const uint4 (&raw)[P::kPasses], float s_inv, const Extent& x, uint32_t* stage) {
    constexpr int NP = P::kPasses;
    const int lane = lane_id();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (!lane_live<P>(x, p)) continue;
        uint32_t t[8];
        quantize8_bits(raw[p], s_inv, t);
        uint2 v;
        v.x = __builtin_amdgcn_perm(__builtin_amdgcn_perm(t[3], t[2], 0x0c0c0400u), __builtin_amdgcn_perm(t[1], t[0], 0x0c0c0400u), 0x05040100u);
        v.y = __builtin_amdgcn_perm(__builtin_amdgcn_perm(t[7], t[6], 0x0c0c0400u), __builtin_amdgcn_perm(t[5], t[4], 0x0c0c0400u), 0x05040100u);
        reinterpret_cast<uint2*>(stage)[piece_index<P, CHAN>(p, lane)] = v;
    }
}

// Table of the 8-bit wrap + zig-zag map, indexed by delta + 256 (delta in [-254, 254]).
__device__ __forceinline__ void fill_zigzag_lut(uint32_t* lut) {
    if (threadIdx.x < 128) {  // four entries per thread
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t b = (4u * threadIdx.x + (uint32_t)e) & 0xFFu;  // (entry - 256) mod 256
            w |= (((b << 1) ^ (0u - (b >> 7))) & 0xFFu) << (8 * e);
        }
        lut[threadIdx.x] = w;
    }
}

// t7 of the lane to the left within the token row; row starts receive `first`.  `carry` is the value
// of lane 63 in the pass before, for a row that continues across the pass boundary (!P::kAligned only).
template <class P>
__device__ __forceinline__ uint32_t left_neighbour(const LanePos& lp, int p, uint32_t first, uint32_t v, uint32_t carry) {
    constexpr int LPR = P::kLpr;
    if (P::kAligned) {
        if (LPR == 16) return dpp<0x111>(first, v);  // row_shr:1, lane 0 of a DPP row keeps `first`
        if (LPR < 16) {
            const uint32_t x = dpp<0x111>(first, v);
            return (lane_id() & (LPR - 1)) == 0 ? first : x;
        }
        const uint32_t x = dpp<0x138>(first, v);  // wave_shr:1 crosses the 16-lane rows
        return (lane_id() & 31) == 0 ? first : x;
    }
    const uint32_t x = dpp<0x138>(carry, v);  // lane 0 has no source lane and keeps `carry`
    return pass_col<P>(lp, p) == 0 ? first : x;
}

// Inclusive prefix sum over the lanes of a token row in pass p.  `carry` is the value this function
// returned at lane 63 in the pass before, for a row that began there (!P::kAligned only).
template <class P>
__device__ __forceinline__ uint32_t row_incl_scan(const LanePos& lp, int p, uint32_t v, uint32_t carry) {
    constexpr int LPR = P::kLpr;
    if (P::kAligned) {
        if (LPR == 16) return row16_incl_scan_dpp(v);
        if (LPR == 32) {
            v = row16_incl_scan_dpp(v);
            return v + dpp<0x142, 0xA>(0, v);  // odd DPP rows add the total of the row before
        }
        const int r = lane_id() & (LPR - 1);
        uint32_t t = dpp<0x111>(0, v);
        v += r >= 1 ? t : 0u;
        t = dpp<0x112>(0, v);
        v += r >= 2 ? t : 0u;
        if (LPR == 4) return v;
        t = dpp<0x114>(0, v);
        return v + (r >= 4 ? t : 0u);
    }
    // rows of LPR lanes begin anywhere: prefix over the whole wave, minus its value just before the
    // row's first lane; a row that began in the pass before adds what it had collected there
    const uint32_t S = wave_incl_scan_dpp(v);
    const int lane = lane_id();
    const int start = lane - (int)pass_col<P>(lp, p);  // first lane of this lane's row (< 0: in the pass before)
    const uint32_t before = (uint32_t)__builtin_amdgcn_ds_bpermute((start > 0 ? start - 1 : 0) << 2, (int)S);
    return start > 0 ? S - before : (start < 0 ? S + carry : S);
}

// Second half of a pass: body offsets, header bits, packing, LDS write.  RUNS = some group of this
// pass may be a run packet (is_run is then meaningful), else every group is literal or all-zero.
template <class P, bool RUNS>
__device__ __forceinline__ void encode_tail(const uint32_t (&u)[8], uint32_t c, uint32_t size, bool is_run, uint32_t qi,
                                            int p, bool live, uint32_t& run, uint32_t* stage, DevState* st) {
    (void)st;  // only the bounds-checking build reads it
    const uint32_t incl = quad_incl_scan_dpp(size);
    const uint32_t off = run + incl - size;  // byte offset of this group's body
    run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    // header: group j of this pass has its code in the quad's lanes; lane 4j+i contributes bit i,
    // so the ballot is the 8 header bytes of the pass (even group in the low nibble)
    const uint64_t hb = __builtin_amdgcn_ballot_w64(((c >> qi) & 1u) != 0);
    if (P::kPartial && p == P::kPasses - 1) {
        // a short page's header ends where its first body begins: bytes, each written by the first lane
        // of the two groups it describes
        const uint32_t lane = (uint32_t)lane_id();
        if (live && (lane & 7u) == 0)
            reinterpret_cast<uint8_t*>(stage)[8 * p + (lane >> 3)] = (uint8_t)(lane < 32 ? (uint32_t)hb >> lane : (uint32_t)(hb >> 32) >> (lane - 32));
    } else if (lane_id() == 0) {
        stage[2 * p] = (uint32_t)hb;
        stage[2 * p + 1] = (uint32_t)(hb >> 32);
    }
    // body: this lane's 8 values are bytes [qi*c, qi*c + c) of the group's little-endian bit string
    uint2 W = pack8_bits(u, c);
    uint32_t B = off + __umul24(qi, c);
    if (RUNS && is_run) {
        W = make_uint2(qi == 0 ? u[0] : 0u, 0u);
        B = off;
    }
    uint32_t* p0 = stage + (B >> 2);
    KVC_CHECK(st, c <= 9 && (B >> 2) + 2 < (uint32_t)Slot<P::kPasses>::kWords && B >= (uint32_t)(P::kPartial ? 8 * (P::kPasses - 1) + 1 : P::kHdr));
    uint32_t d0, d1, d2;
    shl_bytes(W, B, d0, d1, d2);
    atomicOr(p0, d0);
    atomicOr(p0 + 1, d1);
    if (d2) atomicOr(p0 + 2, d2);
}

// One packet group per quad of lanes: each lane brings 8 of its 32 values.  Group statistics over
// the quad (max -> width, run test), then the tail.  p = index of the group's set of 16 (a pass).
template <class P>
__device__ __forceinline__ void encode_groups(const uint32_t (&u)[8], bool RLE, uint32_t c_min, uint32_t qi, int p, bool live,
                                              uint32_t& run, uint32_t* stage, DevState* st) {
    // per-group statistics over the quad of lanes
    uint32_t gmax = max(max(u[0], u[1]), u[2]);
    gmax = max(max(gmax, u[3]), u[4]);
    gmax = max(max(gmax, u[5]), u[6]);
    gmax = max(gmax, u[7]);
    gmax = max(gmax, dpp<0xB1>(0, gmax));
    gmax = max(gmax, dpp<0x4E>(0, gmax));
    // bit length of the group maximum (0 for 0): exponent of its float value
    uint32_t c = max((uint32_t)__builtin_amdgcn_frexp_expf((float)gmax), c_min);
    if (P::kPartial && !live) c = 0;  // a group beyond the page: no header bits, no body (its values are zeros)
    const uint32_t size = c << 2;
    bool cand_any = false;
    uint32_t x = 0;
    if (RLE) {
        // run packet: all 32 values equal and non-zero.  Cheap necessary test first.
        x = (u[0] ^ gmax) | (u[7] ^ gmax);
        cand_any = __builtin_amdgcn_ballot_w64(x == 0 && gmax != 0) != 0;
    }
    if (RLE && cand_any) {
        uint32_t y = x;
#pragma unroll
        for (int k = 1; k < 7; ++k) y |= u[k] ^ gmax;
        y |= dpp<0xB1>(0, y);
        y |= dpp<0x4E>(0, y);
        const bool is_run = (y == 0) && (gmax != 0);
        encode_tail<P, true>(u, is_run ? 9u : c, is_run ? 1u : size, is_run, qi, p, live, run, stage, st);
    } else {
        encode_tail<P, false>(u, c, size, false, qi, p, live, run, stage, st);
    }
}

// Byte offset, inside a page, of the 16 bytes a lane handles in pass p, as a wave-uniform part plus a
// per-lane part that stays in 32 bits (the layout setter bounds the row stride): a page access is then a
// wave-uniform 64-bit base plus a 32-bit lane offset.  Row-major deal: lane l of pass p holds token row
// (64p + l) / (D/8), channels 8 * ((64p + l) mod (D/8)) .. +7; with contiguous rows a pass is one 1 KB
// run.  When D divides 512 the lane part is the same in every pass.  Mode 5 (CHAN, see piece_index):
// lane 4l + r takes token 4 (p mod 4) + r of octet 16 (p div 4) + l.
template <class P, bool CHAN>
__device__ __forceinline__ int64_t pass_base_off(const Geometry& g, int p) {
    if (CHAN) return (int64_t)(p & 3) * 4 * g.row_stride * 2 + (P::kD == 64 ? 0 : (p >> 2) * 256);
    return (int64_t)((p * 64) / P::kLpr) * g.row_stride * 2;  // the whole rows before the pass
}
template <class P, bool CHAN>
__device__ __forceinline__ uint32_t pass_lane_off(const Geometry& g, const LanePos& lp, int p) {
    if (CHAN) return lp.off0_chan;
    if (P::kAligned) return lp.off0;
    const uint32_t c = lp.col0 + (uint32_t)((p * 64) % P::kLpr);  // the pass begins this far into a row
    const bool wrap = c >= (uint32_t)P::kLpr;
    return ((lp.row0 + (wrap ? 1u : 0u)) * (uint32_t)g.row_stride + (wrap ? c - P::kLpr : c) * 8u) * 2u;
}

// A page's loads, `src` its first element.  Nothing here is behind a branch: the loads of a batch of pages are then in
// flight together and each page waits for its own only.  (Lanes beyond a short page read the 16 bytes that begin
// the last pass's first row, and hold zeros.)
template <class P, bool CHAN>
__device__ __forceinline__ void load_page(const EncodeArgs& a, const char* src, const LanePos& lp, uint4 (&raw)[P::kPasses]) {
    const Extent x = page_extent<P>(a.g);
#pragma unroll
    for (int p = 0; p < P::kPasses; ++p) {
        const bool live = lane_live<P>(x, p);
        const uint32_t off = pass_lane_off<P, CHAN>(a.g, lp, p);
        raw[p] = load_stream(reinterpret_cast<const uint4*>(src + pass_base_off<P, CHAN>(a.g, p) + (live ? off : 0u)));
    }
}
// ... once they have arrived: lanes beyond a short page hold zeros
template <class P>
__device__ __forceinline__ void clear_beyond(const Extent& x, uint4 (&raw)[P::kPasses]) {
    if (!P::kPartial) return;
    constexpr int p = P::kPasses - 1;
    const uint32_t keep = lane_live<P>(x, p) ? ~0u : 0u;
    raw[p] = make_uint4(raw[p].x & keep, raw[p].y & keep, raw[p].z & keep, raw[p].w & keep);
}

// Mode 5: the packets of a page whose 128-bit pieces were dealt to the lanes as piece_index<P, true> says;
// every group holds one pair of neighbouring channels over the 16 tokens.
template <class P>
__device__ __forceinline__ void pack_channel_pairs(const uint4 (&raw)[P::kPasses], float s_inv, uint32_t& run, uint32_t* stage,
                                                   const uint8_t* lut, DevState* st) {
    static_assert(P::kChan, "mode 5 is built for 16-token pages of 64, 128 or 256 channels");
    constexpr int NP = P::kPasses;
    const int lane = lane_id();
    const uint32_t qi = (uint32_t)lane & 3u;
    if constexpr (P::kD == 64) {
        // Eight octets: a lane holds tokens 8h + r and 8h + 4 + r of its octet (two passes), its partner 32
        // lanes away the other eight tokens' share.  Of the octet's four channel pairs the lane packs pairs h
        // and 2 + h (group sets 0 and 1), the partner the other two; each hands the other the four values it
        // holds of the other's pair.  Value index inside a packet: 2 * (token div 4) + (channel mod 2), token
        // div 4 = 2h + p.
        static_assert(NP == 2, "sixteen tokens of eight octets are two passes");
        const bool hi = lane >= 32;
        uint32_t uu[2][8];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint32_t t[8];
            quantize8_bits(raw[p], s_inv, t);
#pragma unroll
            for (int k = 0; k < 8; ++k) uu[p][k] = lut[t[k] - (kMagicBits + 256u * (uint32_t)k - 256u)];
        }
#pragma unroll
        for (int sset = 0; sset < 2; ++sset) {
            uint32_t u[8];
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const uint32_t lo_pair = uu[p][4 * sset + e], hi_pair = uu[p][4 * sset + 2 + e];  // pairs 2 sset, 2 sset + 1
                    const uint32_t mine = hi ? hi_pair : lo_pair;
                    const uint32_t got = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)(hi ? lo_pair : hi_pair));
                    u[2 * p + e] = hi ? got : mine;
                    u[4 + 2 * p + e] = hi ? mine : got;
                }
            encode_groups<P>(u, true, 0u, qi, sset, true, run, stage, st);
        }
    } else {
        // Sixteen or 32 octets: the four passes of a run of 16 octets are quantized and mapped first; group
        // set j of the run then takes channels 2j, 2j + 1 of each of them: the quad's 32 values are one
        // channel pair over the 16 tokens.
#pragma unroll
        for (int h = 0; h < NP / 4; ++h) {
            uint32_t uu[4][8];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                uint32_t t[8];
                quantize8_bits(raw[4 * h + p], s_inv, t);
#pragma unroll
                for (int k = 0; k < 8; ++k) uu[p][k] = lut[t[k] - (kMagicBits + 256u * (uint32_t)k - 256u)];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t u[8];
#pragma unroll
                for (int m = 0; m < 8; ++m) u[m] = uu[m >> 1][2 * j + (m & 1)];
                encode_groups<P>(u, true, 0u, qi, 4 * h + j, true, run, stage, st);
            }
        }
    }
}

// Encode one page (already in registers) into the LDS slot `stage`.  The requested mode is the
// compile-time SCHEME when that is >= 0 (one mode for the whole launch: its branches fold away), else
// the wave-uniform run-time value: any of modes 0..4 (SCHEME -1), or any of 0..5 (SCHEME -2, built for
// the page shapes that have mode 5; the page must then have been loaded in the deal of its mode).
template <class P, int SCHEME>
__device__ __forceinline__ PageResult encode_page(const uint4 (&raw)[P::kPasses], const LanePos& lp, const Extent& x, int scheme_rt,
                                                 uint32_t* stage, const uint8_t* lut, DevState* st) {
    const int scheme = SCHEME >= 0 ? SCHEME : scheme_rt;
    constexpr int kE = P::kE, NP = P::kPasses;
    constexpr bool kMayChan = SCHEME == KVC_MODE_CHAN || SCHEME == kSchemeAny;
    const bool chan = SCHEME == KVC_MODE_CHAN || (SCHEME == kSchemeAny && scheme == KVC_MODE_CHAN);
    const bool RLE = scheme != KVC_MODE_DELTA;  // zero-run and run packets (modes 3 and 4)
    const bool no_delta = scheme == KVC_MODE_PACK;
    const uint32_t c_min = RLE ? 0u : 1u;  // without run packets an all-zero group is a 1-bit literal
    const int lane = lane_id();
    const uint32_t qi = (uint32_t)lane & 3u;

    // scaling: max |x|, two values per dword; the magnitudes compare as integers across the lanes
    half2v mh = {(_Float16)0.0f, (_Float16)0.0f};
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        mh = max_magnitude(mh, raw[p].x);
        mh = max_magnitude(mh, raw[p].y);
        mh = max_magnitude(mh, raw[p].z);
        mh = max_magnitude(mh, raw[p].w);
    }
    const uint32_t m2 = __builtin_bit_cast(uint32_t, mh) & 0x7FFF7FFFu;
    const uint32_t m = wave_max_dpp(max(m2 & 0xFFFFu, m2 >> 16));
    PageResult r;
    if (scheme == KVC_MODE_RAW || m >= 0x7C00u) {  // requested, or NaN/Inf present: bypass
        r.n16 = x.E >> 3;
        r.mode = KVC_MODE_RAW;
        r.scale = 0.0f;
        return r;
    }
    float s = 0.0f, s_inv = 0.0f;
    if (m != 0) {
        const PageScale ps = page_scale(m);
        s = ps.s;
        s_inv = ps.s_inv;
    }
    r.scale = s;
    auto codes_to_stage = [&]() {  // the plain INT8 payload, from whichever deal the lanes hold
        if constexpr (kMayChan) {
            if (chan) {
                store_codes<P, true>(raw, s_inv, x, stage);
                return;
            }
        }
        store_codes<P, false>(raw, s_inv, x, stage);
    };
    if (scheme == KVC_MODE_INT8) {
        codes_to_stage();
        r.n16 = x.E >> 4;
        r.mode = KVC_MODE_INT8;
        return r;
    }
    // bodies are OR-ed into the slot, and the zero padding is part of the payload
#pragma unroll
    for (int z = 0; z < P::kRounds; ++z)
        if (kE % 1024 == 0 || lane + 64 * z < kE / 16) reinterpret_cast<uint4*>(stage)[lane + 64 * z] = make_uint4(0, 0, 0, 0);
    wave_sync();

    uint32_t run = x.hdr;  // payload bytes so far (wave-uniform)
    bool packed_by_pairs = false;
    if constexpr (kMayChan) {
        if (chan) {
            pack_channel_pairs<P>(raw, s_inv, run, stage, lut, st);
            packed_by_pairs = true;
        }
    }
    if (!packed_by_pairs) {
        uint32_t carry = kMagicBits - 256u;  // last value of the pass before, for a row that continues
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            uint32_t t[8];
            quantize8_bits(raw[p], s_inv, t);
            // delta along the channel index, plus 256; the first column of a token row has no left
            // neighbour and is kept verbatim (q - 0).  Then wrap + zig-zag by table.
            uint32_t u[8];
            if (no_delta) {  // mode 4: the table is indexed by q + 256
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = lut[t[k] - (kMagicBits + 256u * (uint32_t)k - 256u)];
            } else {
                const uint32_t prev = left_neighbour<P>(lp, p, kMagicBits - 256u, t[7] - 2048u, carry);
                if (!P::kAligned) carry = (uint32_t)__builtin_amdgcn_readlane((int)(t[7] - 2048u), 63);
                KVC_CHECK(st, t[0] - prev < 512u && t[1] - t[0] < 512u && t[7] - t[6] < 512u);
                u[0] = lut[t[0] - prev];
#pragma unroll
                for (int k = 1; k < 8; ++k) u[k] = lut[t[k] - t[k - 1]];
            }
            const bool live = lane_live<P>(x, p);
            if (P::kPartial && p == NP - 1) {  // lanes beyond the page hold no values
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = live ? u[k] : 0u;
            }
            encode_groups<P>(u, RLE, c_min, qi, p, live, run, stage, st);
        }
    }
    const uint32_t n = (run + 15u) & ~15u;
    wave_sync();
    if (n >= x.E) {  // packing did not beat plain INT8
        codes_to_stage();
        r.n16 = x.E >> 4;
        r.mode = KVC_MODE_INT8;
    } else {
        r.n16 = n >> 4;
        r.mode = (uint32_t)scheme;
    }
    return r;
}

// Encoder launch shape for large calls, by passes per page: waves per workgroup, pages per wave, pages a wave holds in
// registers at once.  A workgroup takes one atomic on the pool cursor, and the cursor's line serves one every 13 ns
// whoever asks: with 64 KB of input per workgroup a launch at full bandwidth keeps it busy four fifths of the time,
// and half of that makes it the bound (a million pages of 16 x 128: 32 KB per workgroup 1725 us, 64 KB 1055, 80 to 128
// KB 970 to 1000).  The payloads wait in LDS meanwhile, half a byte per byte, so 160 KB per workgroup and more leave
// a compute unit one workgroup and nothing to overlap its phases with (1475 us).  Between those the shapes are the
// best of a sweep; compress, us, 64 KB shape -> this one: 16 x 64 272 -> 260, 16 x 96 420 -> 382, 16 x 128 1055 -> 970,
// 32 x 96 389 -> 371, 16 x 224 509 -> 432, 16 x 256 532 -> 504 (1 KB pages: 96 and 128 KB are slower, 145 -> 172).  The
// instantiations that read the mode at run time need more registers and have shapes of their own (INT8 at 16 x 128
// 272 -> 253, 16 x 96 421 -> 388, 32 x 96 381 -> 368, 24 x 96 135 -> 124, 16 x 224 511 -> 475).
struct EncShape {
    int waves, ppw, ring;
};
constexpr EncShape enc_large(int np, int scheme) {
    constexpr EncShape fixed[9] = {{0, 0, 0}, {8, 8, 8}, {8, 5, 5}, {8, 3, 3}, {4, 5, 5}, {8, 2, 2}, {8, 2, 2}, {8, 2, 2}, {8, 2, 1}};
    constexpr EncShape run_time[9] = {{0, 0, 0}, {8, 8, 8}, {4, 8, 8}, {4, 6, 3}, {8, 3, 3}, {8, 2, 2}, {8, 2, 2}, {4, 3, 1}, {4, 2, 1}};
    return scheme >= 0 ? fixed[np] : run_time[np];
}
constexpr int enc_ring(int np, int ppw, int scheme) { return ppw <= enc_large(np, scheme).ring ? ppw : enc_large(np, scheme).ring; }

// (four waves per SIMD is about what the LDS slots allow anyway: keep the instantiations within 128 VGPRs; where the
// slots allow three -- four-pass pages with the mode fixed --, the channel-pair encoder at D = 256 holds 32 mapped
// values beside the page, and the run-time-scheme encoders of seven- and eight-pass pages whose rows cross passes or
// whose last pass may be short would spill at four)
template <class P, int SCHEME>
constexpr int enc_min_waves() {
    return ((P::kPasses == 4 && SCHEME >= 0) || (P::kD == 256 && (SCHEME == KVC_MODE_CHAN || SCHEME == kSchemeAny)) || (P::kPasses >= 7 && (!P::kAligned || P::kPartial) && SCHEME < 0)) ? 3 : 4;
}
// A page task as it is parked in LDS: what a later turn of the loop, or the end of the kernel, needs to know of it.
struct EncPlace {
    uint64_t di;
    int32_t sb;
    uint32_t pg;
    int scheme;
    uint32_t w;  // once encoded: n16 | mode << 16 ...
    float s;     // ... and the scale
};

// 8 KB pages, large-call shapes, calls of at most this many pages: the tasks are dealt to the workgroups in order and not
// by eighths.  (An eighth is then often a power of two away from the next, and the XCDs presumably meet at the same memory
// channels: pages of 7.5 KB and less show nothing of it.)  Compress, us, by eighths -> in order: mode 4, 8,192 pages 27.5 ->
// 26.3, 12,288 42.5 -> 38.8, 32,768 86.7 -> 84.3; mode 3, 16,384 pages 43.4 -> 40.9; mode 5, 12,288 pages 35.3 -> 33.2.  On
// larger calls the encoder gains less than the decoder loses on the pool it leaves (2 to 3 % from 131,072 pages on).
constexpr int kEncInOrder8Kb = 32768;

// LDS words of a wave's payloads: they follow one another as the pages are encoded, an encoded page holds at most the 512
// bytes per pass of its INT8 form, and the one at work has a whole slot.
constexpr int enc_stage_words(int np, int ppw) { return (ppw - 1) * np * 128 + ((np * 520 + 16 + 15) / 16) * 4; }

template <class P, int WAVES, int PPW, int SCHEME>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(enc_min_waves<P, SCHEME>()))) void k_compress(EncodeArgs a) {
    constexpr int NP = P::kPasses;
    constexpr int kMaxMode = SCHEME == kSchemeAny ? KVC_MODE_CHAN : KVC_MODE_PACK;  // what a per-block request may ask for
    constexpr int kRing = enc_ring(NP, PPW, SCHEME);
    constexpr bool kUniform = PPW == 1;  // one page per wave: resolved on the scalar unit
    constexpr bool kSmall = PPW == 1 && WAVES == 4;  // calls of up to 512 pages: they copy their pages in plain rounds too (see below)
    static_assert(PPW % kRing == 0 && PPW <= 16, "the loop handles pages in groups of kRing; a row of lanes scans them");
    __shared__ __align__(16) uint32_t s_stage[WAVES][enc_stage_words(NP, PPW)];
    __shared__ uint32_t s_lut[128];
    __shared__ uint32_t s_total[WAVES];  // units of each wave's payloads; kHasRaw: raw pages among them
    __shared__ unsigned long long s_base;  // its span of the pool begins at this unit; kKept: and is to stay in the last-level cache
    constexpr unsigned long long kKept = 1ull << 63;
    constexpr uint32_t kHasRaw = 1u << 24;
    static_assert(WAVES * PPW * NP * 64 < (1 << 24) && WAVES < 128, "the sum over a workgroup keeps both parts apart");
    __shared__ EncPlace s_place[WAVES * PPW];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint8_t* lut = reinterpret_cast<const uint8_t*>(s_lut);
    uint32_t* const staged = s_stage[wave];  // the wave's payloads, one after the other
    const Extent x = page_extent<P>(a.g);
    const LanePos lp = lane_pos<P>(a.g);
    constexpr unsigned kInOrder = P::kPasses == 8 && !P::kPartial && PPW > 1 ? kEncInOrder8Kb / (WAVES * PPW) : 0;  // workgroups
    const int64_t t0 = ((int64_t)(kInOrder && gridDim.x <= kInOrder ? blockIdx.x : task_block_index()) * WAVES + wave) * PPW;
    const EncLanes L = kUniform ? enc_locate(a, t0 < a.n_pages, (uint32_t)t0, kMaxMode)
                                : enc_locate(a, lane < PPW && t0 + lane < a.n_pages, (uint32_t)t0 + (uint32_t)lane, kMaxMode);
    const uint32_t ok = kUniform ? (L.ok ? 1u : 0u) : (uint32_t)__builtin_amdgcn_ballot_w64(L.ok);
    if (lane < PPW) s_place[wave * PPW + lane] = EncPlace{L.di, L.sb, L.pg, L.scheme, 0u, 0.0f};  // (not kept in registers meanwhile)
    wave_sync();
    uint32_t total = 0;  // payload units of the wave's pages,
    uint32_t held = 0;   // and those of them that are staged (raw payloads are not)
    const int any = __builtin_ctz(ok | 0x10000u);  // a page that exists: the loads of those that do not read it again
    // the deal of the page to the lanes follows the mode requested for it
    constexpr bool kParked = kRing < PPW;  // pages are loaded while others are encoded
    auto scheme_of = [&](int i) { return kParked ? (int)wave_uniform((int32_t)s_place[wave * PPW + i].scheme) : (int)of_lane<kUniform>((uint32_t)L.scheme, i); };
    auto load = [&](int i, uint4 (&raw)[NP]) {
        const int from = (ok >> i) & 1u ? i : any;
        const EncPlace& parked = s_place[wave * PPW + from];
        const int32_t sb = kParked ? wave_uniform(parked.sb) : (int32_t)of_lane<kUniform>((uint32_t)L.sb, from);
        const int32_t pg = kParked ? wave_uniform((int32_t)parked.pg) : (int32_t)of_lane<kUniform>(L.pg, from);
        const int64_t off = page_base(a.g, sb, pg);
        const char* src = reinterpret_cast<const char*>(a.cache) + off * 2;
        if constexpr (SCHEME == kSchemeAny) {
            if (scheme_of(i) == KVC_MODE_CHAN)
                load_page<P, true>(a, src, lp, raw);
            else
                load_page<P, false>(a, src, lp, raw);
        } else {
            load_page<P, SCHEME == KVC_MODE_CHAN>(a, src, lp, raw);
        }
    };
    auto encode = [&](int i, uint4 (&raw)[NP]) {
        if (((ok >> i) & 1u) == 0) return;
        clear_beyond<P>(x, raw);
        const PageResult r = encode_page<P, SCHEME>(raw, lp, x, scheme_of(i), staged + 4u * held, lut, a.st);
        if (lane == 0) {
            s_place[wave * PPW + i].w = r.n16 | (r.mode << 16);
            s_place[wave * PPW + i].s = r.scale;
        }
        total += r.n16;
        held += r.mode == KVC_MODE_RAW ? 0u : r.n16;
    };
    // The register sets take turns (the inner loop is unrolled, so every index is a constant): nothing is copied
    // between them, and up to kRing pages' loads are in flight.
    uint4 raw[kRing][NP];
    if (ok) {
#pragma unroll
        for (int j = 0; j < kRing - 1; ++j) load(j, raw[j]);
    }
    fill_zigzag_lut(s_lut);
    __syncthreads();
    if (ok) {
#pragma unroll 1
        for (int i = 0; i < PPW; i += kRing) {
#pragma unroll
            for (int j = 0; j < kRing; ++j) {
                const int next = i + j + kRing - 1;
                if (kRing == PPW ? j == 0 : next < PPW) load(kRing == PPW ? kRing - 1 : next, raw[(j + kRing - 1) % kRing]);
                encode(i + j, raw[j]);
            }
        }
    }
    // One atomic on the pool cursor reserves a contiguous span for all pages of the workgroup.
    if (lane == 0) s_total[wave] = total | (held != total ? kHasRaw : 0u);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sum = 0;  // (units of all waves, and above them how many have raw pages)
#pragma unroll
        for (int k = 0; k < WAVES; ++k) sum += s_total[k];
        const uint32_t all = sum % kHasRaw;
        const unsigned long long base = all ? atomicAdd(&a.st->cursor16, (unsigned long long)all) : 0ull;
        if (base + all > a.pool_units) atomicOr(&a.st->status, KVC_ST_POOL_FULL);
        s_base = sum < kHasRaw && base < a.kept_units ? base | kKept : base;
    }
    __syncthreads();
    if (ok == 0) return;
    // lane i: where page i's payload goes; pages that do not fit become INVALID
    uint32_t before = 0;  // units of the waves before this one
#pragma unroll
    for (int k = 0; k < WAVES - 1; ++k) before += k < wave ? s_total[k] : 0u;
    before %= kHasRaw;
    wave_sync();
    const EncPlace& own = s_place[wave * PPW + min(lane, PPW - 1)];
    const uint32_t w_own = lane < PPW ? own.w : 0u;  // lane i: page i's
    const uint32_t n_own = w_own & 0xFFFFu;
    const uint64_t off16 = s_base % kKept + before + (kUniform ? 0u : row16_incl_scan_dpp(n_own) - n_own);
    const bool fits = off16 + n_own <= a.pool_units;
    if (lane < 32 && ((ok >> (lane & 31)) & 1u)) {
        const uint64_t off = off16 * 16u;
        reinterpret_cast<uint4*>(a.desc)[own.di] =
            fits ? make_uint4((uint32_t)off, (uint32_t)(off >> 32), __float_as_uint(own.s), w_own) : make_uint4(0u, 0u, 0u, (uint32_t)KVC_MODE_INVALID << 16);
    }
    // The staged payloads are one run in LDS and, where the wave has no raw pages, in the pool.  That is copied as one, and by lines
    // of the pool: every round of lanes but the first and the last stores eight whole lines, and a line belongs to one store unless
    // it is shared with another wave.  (Page by page, each with rounds of its own, every page split a line in two stores,
    // which the streaming hint often sends to the memory one by one.  Compress, us: half a million pages of 16 x 128, mode
    // 5, 484 -> 477, a million of mode 3 973 -> 966, 524,288 of 16 x 96 378 -> 368, of 16 x 64 257 -> 250, of 16 x 32 by
    // block ids 151 -> 142; up to 16,384 pages the same.)  A wave of one page does without the lines.
    const uint32_t unfit = ok & (uint32_t)__builtin_amdgcn_ballot_w64(!fits);  // (the wave's last pages, if any)
    const uint32_t raws = ok & (uint32_t)__builtin_amdgcn_ballot_w64(w_own >> 16 == KVC_MODE_RAW);
    const uint64_t base16 = of_lane<false>(off16, 0);
    auto copy_out = [&](auto aux, uint64_t to16, uint32_t n) {  // n units from the beginning of the stage to unit `to16` of the pool
        if (n == 0) return;
        const uint4* src = reinterpret_cast<const uint4*>(staged);
        KVC_CHECK(a.st, to16 + n <= a.pool_units && n * 4u <= (uint32_t)enc_stage_words(NP, PPW));
        const uint32_t skew = kUniform ? 0u : (uint32_t)to16 & 7u;  // units of the first line that are not the wave's
        const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(a.pool + (to16 - skew) * 16u, 0, (int)((skew + n) * 16u), 0x00020000);
        constexpr int kAhead = PPW * 32 * NP >= 256 ? 4 : (PPW * 32 * NP + 63) / 64;
        for (uint32_t u0 = 0; u0 < skew + n; u0 += 64u * kAhead) {
            uint4v v[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const uint4 t = src[min((uint32_t)max((int)(u0 + lane + 64u * k - skew), 0), n - 1u)];
                v[k].x = t.x; v[k].y = t.y; v[k].z = t.z; v[k].w = t.w;
            }
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {  // (units beyond the last are out of the resource's range, and so are those before the first made to be: not stored)
                uint32_t at = (u0 + lane + 64u * k) * 16u;
                if (k == 0) at = u0 + lane < skew ? ~15u : at;
                __builtin_amdgcn_raw_buffer_store_b128(v[k], dst, (int)at, 0, decltype(aux)::value);
            }
        }
    };
    // (One answer for a workgroup, and no where it holds raw pages: those are read again and stored plainly, they need the cache
    // for themselves.  Compress / compress and decompress, us, every payload stored past the cache, those of clean waves kept, those
    // of clean workgroups: 256 MiB of 16 x 64, every second page raw, 104 / 180, 103 / 182, 103 / 181, of 16 x 256 116 / 203,
    // 119 / 217, 116 / 203; one page in 64 raw 75 / 145, 73 / 130, 74 / 136.)
    const bool kept = wave_uniform((int32_t)(s_base >> 32)) < 0;
    // (Calls of up to 512 pages, a page a wave, take every instruction in a chain: with the general copy, twice over, reset and compress of 64
    // pages, nothing kept, 16 x 32 take 4.5 us in mode 1 and 16 x 128 4.8, 4.45 and 4.75 with the plain rounds below; 5.1 with the general copy, kept.)
    if (!kSmall && raws == 0) {
        const uint32_t n = unfit ? (uint32_t)(of_lane<false>(off16, __builtin_ctz(unfit)) - base16) : total;
        if (kept)
            copy_out(std::integral_constant<int, 16>{}, base16, n);  // sc1: through the L2, to stay in the last-level cache
        else
            copy_out(std::integral_constant<int, 2>{}, base16, n);  // nt
        return;
    }
    uint32_t from = 0;
#pragma unroll 1
    for (int i = 0; i < PPW; ++i) {
        if (((ok & ~unfit) >> i & 1u) == 0) continue;
        const uint32_t w = of_lane<false>(w_own, i), n16 = w & 0xFFFFu;
        const uint64_t to16 = of_lane<false>(off16, i);
        if (w >> 16 != KVC_MODE_RAW) {
            // page by page, in plain rounds: the rounds by lines cost more than they save on so short runs (compress, us, 256 MiB
            // with every second page raw: 16 x 64 134 -> 104, 16 x 128 134 -> 117; 1 GiB of 16 x 32, one in 16: 327 -> 290)
            KVC_CHECK(a.st, to16 + n16 <= a.pool_units && (from + n16) * 4u <= (uint32_t)enc_stage_words(NP, PPW));
            uint4* to = reinterpret_cast<uint4*>(a.pool) + to16;
            const uint4* src = reinterpret_cast<const uint4*>(staged) + from;
            if (kSmall && kept) {
                const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(to, 0, (int)(n16 * 16u), 0x00020000);
#pragma unroll
                for (int z = 0; z < P::kRounds; ++z) {
                    if ((uint32_t)lane + 64u * z >= n16) continue;
                    const uint4 t = src[lane + 64 * z];
                    const uint4v v = {t.x, t.y, t.z, t.w};
                    __builtin_amdgcn_raw_buffer_store_b128(v, dst, (lane + 64 * z) * 16, 0, 16);
                }
                return;
            }
#pragma unroll
            for (int z = 0; z < P::kRounds; ++z)
                if ((uint32_t)lane + 64u * z < n16) store_stream(to + lane + 64 * z, src[lane + 64 * z]);
            from += n16;
            continue;
        }
        // the payload is the dense page
        KVC_CHECK(a.st, to16 + n16 <= a.pool_units);
        uint4* dst = reinterpret_cast<uint4*>(a.pool) + to16;
        const EncPlace pl = s_place[wave * PPW + i];
        const uint16_t* srcp = a.cache + page_base(a.g, (int64_t)wave_uniform(pl.sb), wave_uniform((int32_t)pl.pg));
        for (uint32_t o = (uint32_t)lane; o < n16; o += 64) dst[o] = *reinterpret_cast<const uint4*>(srcp + elem_off(a.g, (int)o * 8));
    }
}

// ---------------------------------------------------------------------------------- decode

// dequantize: x = fp16(fp32(q) * s).  b = (q + 128) mod 256 sits in the low byte of pb; the fused
// b*s - 128*s rounds q*s once to binary32 (128*s is exact), then one rounding to FP16, for two values at once.  (The
// compiler would rather fuse the product with the conversion, v_fma_mixlo/hi_f16; those issue once in 8.5 cycles each,
// v_fma_f32 in 2.6 and v_cvt_pk_f16_f32, which converts two, in 4.3: 17 against 9.6 cycles per pair.)
__device__ __forceinline__ uint4 dequant8_biased(const uint32_t pb[8], float s, float neg128s) {
    half2v h[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float2v f = {__builtin_fmaf((float)(pb[2 * k] & 0xFFu), s, neg128s), __builtin_fmaf((float)(pb[2 * k + 1] & 0xFFu), s, neg128s)};
        asm("" : "+v"(f.x), "+v"(f.y));
        h[k] = __builtin_convertvector(f, half2v);
    }
    return make_uint4(__builtin_bit_cast(uint32_t, h[0]), __builtin_bit_cast(uint32_t, h[1]),
                      __builtin_bit_cast(uint32_t, h[2]), __builtin_bit_cast(uint32_t, h[3]));
}

// Stores of the decoder's output at base + off (wave-uniform) + lane_off.  They write through the XCD's L2 (device scope)
// and are not kept there.  Under the prefetch window a block is thereby published by waiting for its stores, without a
// write-back of the whole L2; and every launch is faster so: written back in the L2's own time instead, the pages that
// 8,000 waves are writing at once reach the memory in no order (a million pages of 16 x 128, us: 1025 -> 1013, half a
// million of mode 5 515 -> 503, 262,144 raw pages 381 -> 371; without the streaming hint 1063).
__device__ __forceinline__ void store_out(char* base, int64_t off, uint32_t lane_off, const uint4& v) {
    uint4v w;
    w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    // aux: 16 = sc1, device scope; 2 = nt.  The uniform offset goes into the resource and not into the store's scalar
    // offset: a store of more than 64 bits needs a wait state before its data registers are written again, and
    // with a scalar offset the compiler leaves it out, taking the store to be safe -- on this chip it is not (one
    // page in a hundred came out with the first dword of some lanes replaced by what was computed next).
    __builtin_amdgcn_raw_buffer_store_b128(w, __builtin_amdgcn_make_buffer_rsrc(base + off, 0, -1, 0x00020000), (int)lane_off, 0, 16 | 2);
}
__device__ __forceinline__ void zero_out(uint16_t* dst, const Geometry& g) {
    for (int o = lane_id(); o < (g.E >> 3); o += 64)
        store_out(reinterpret_cast<char*>(dst), 0, (uint32_t)elem_off(g, o * 8) * 2u, make_uint4(0u, 0u, 0u, 0u));
}

// What the header scan leaves for a packet group: where its body begins in the slot, its code c, and the byte mask that
// keeps the upper c - 1 bits of a c-bit field.
struct GroupInfo {
    uint32_t at;    // body offset << 12 | c << 8 | 4 (c - 1) mod 32
    uint32_t high;  // 2^(c-1) - 1 in every byte
};
__device__ __forceinline__ GroupInfo group_pack(uint32_t off, uint32_t c) {
    GroupInfo g;
    g.at = (off << 12) | (c << 8) | (((c - 1u) << 2) & 31u);
    g.high = 0x01010101u * ((1u << ((c - 1u) & 7u)) - 1u);
    return g;
}

// (m & a) | (~m & b), as the instruction of this chip that takes half the time of a bit-field insert
__device__ __forceinline__ uint32_t select_bits(uint32_t m, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA); }

// Four c-bit fields (the low 4c bits of x, 1 <= c <= 8) to the four bytes of a dword, each undone from its zig-zag code
// and biased by 128 (mod 256).  sh = 8 - c.  Four values at a time, because the decoder of a whole cache keeps the
// vector units busy two thirds of its time and a transfer engine of the prefetch window waits for them: a field, its
// sign and the sum took 2.9 instructions of 4.4 cycles per value one by one, these take 2 of mostly 2.5.
__device__ __forceinline__ uint32_t fields_to_bytes(uint32_t x, uint32_t sh, uint32_t high) {
    x = select_bits(0x0000FFFFu, x, x << (sh + sh));  // fields 2 and 3 to the upper half
    x = select_bits(0x00FF00FFu, x, x << sh);         // fields 1 and 3 to the odd bytes (a byte's bits above c are whatever followed)
    const uint32_t sign = 0x80808080u - (x & 0x01010101u);  // per byte 0x80, or 0x7F from an odd code: its sign, with the bias
    return ((x >> 1) & high) ^ sign;
}

// This lane's 8 values of its quad's packet in group set p, read from the staged payload and undone from their zig-zag
// codes: value k is byte k of the two dwords, plus 128 (mod 256).  SPECIAL: the page has zero-run or run packets (few
// pages do, and the others are decoded without the tests for them).
template <int NP, bool SPECIAL>
__device__ __forceinline__ void unpack8(const DecodeArgs& a, const uint32_t* stage, const GroupInfo& g, uint32_t hdr, uint32_t (&w)[2]) {
    (void)hdr;
    (void)a;  // only the bounds-checking build reads them
    const uint32_t qi = (uint32_t)lane_id() & 3u;
    uint32_t c = (g.at >> 8) & 15u;
    const uint32_t goff = g.at >> 12;
    uint32_t high = g.high;
    uint32_t B = goff + __umul24(qi, c);
    if (SPECIAL && c == 9) B = goff;
    const uint32_t* p0 = stage + (B >> 2);
    KVC_CHECK(a.st, (B >> 2) + 2 < (uint32_t)Slot<NP>::kWords && B >= hdr);  // bodies start after the header bytes
    const uint32_t d0 = p0[0], d1 = p0[1], d2 = p0[2];
    uint32_t lo = __builtin_amdgcn_alignbyte(d1, d0, B);  // (a byte shift is taken mod 4, a bit shift mod 32)
    const uint32_t up = __builtin_amdgcn_alignbyte(d2, d1, B);
    // values 0..3 are bits 0 .. 4c - 1 of (up : lo), values 4..7 the 4c bits after those: shifted down by 4, then by 4c - 4
    uint32_t hi = __builtin_amdgcn_alignbit(up >> 4, __builtin_amdgcn_alignbit(up, lo, 4u), g.at);
    if (SPECIAL) {
        if (c == 9) {  // run packet: the body byte, 32 times
            lo = __builtin_amdgcn_perm(lo, lo, 0u);
            hi = lo;
            c = 8;
            high = 0x7F7F7F7Fu;
        } else if (c == 0) {  // zero-run packet
            lo = 0;
            hi = 0;
        }
    }
    const uint32_t sh = 8u - c;
    w[0] = fields_to_bytes(lo, sh, high);
    w[1] = fields_to_bytes(hi, sh, high);
}

template <class P>
__device__ __forceinline__ bool is_packed_mode(uint32_t mode) {
    return mode == KVC_MODE_DELTA || mode == KVC_MODE_RLE || mode == KVC_MODE_PACK || (P::kChan && mode == KVC_MODE_CHAN);
}

// Lane-wise second half of the resolution: ask for the descriptor, and -- once it is there -- validate it against the pool
// and the page geometry.  Sticky status bits of bad indices and descriptors are set in the second part.
struct DecDue {
    uint64_t di;                   // descriptor index
    bool stray, wanted, readable;  // output block out of range; a page is due; its descriptor exists
};
__device__ __forceinline__ DecDue dec_due(const DecodeArgs& a, const DecPlace& t) {
    const bool placed = t.live && t.db >= 0 && t.db < a.n_out_blocks;
    DecDue r;
    r.di = (uint64_t)t.pb * (uint64_t)a.g.ppb + t.pg;
    r.stray = t.live && t.db >= 0 && !placed;
    r.wanted = placed && (t.bad_index || t.pb >= 0);
    r.readable = r.wanted && !t.bad_index && r.di < a.n_desc;
    return r;
}
__device__ __forceinline__ uint4 dec_ask(const DecodeArgs& a, const DecPlace& t) {
    const DecDue due = dec_due(a, t);
    uint4 dw = make_uint4(0u, 0u, 0u, 0u);
    if (due.readable) dw = reinterpret_cast<const uint4*>(a.desc)[due.di];
    return dw;
}
template <class P>
__device__ __forceinline__ DecLanes dec_check(const DecodeArgs& a, const DecPlace& t, const uint4& dw) {
    const Extent x = page_extent<P>(a.g);
    const DecDue due = dec_due(a, t);
    DecLanes r;
    r.db = t.db;
    r.pg = t.pg;
    r.off = (uint64_t)dw.x | ((uint64_t)dw.y << 32);
    r.s = __uint_as_float(dw.z);
    const uint32_t n16 = dw.w & 0xFFFFu, mode = (dw.w >> 16) & 0xFFu;
    const bool raw = mode == KVC_MODE_RAW;
    const bool in_pool = (r.off & 15u) == 0 && (r.off >> 4) + n16 <= a.pool_units;
    const bool sized = raw ? n16 == x.E >> 3 : mode == KVC_MODE_INT8 ? n16 == x.E >> 4 : is_packed_mode<P>(mode) && n16 * 16u >= x.hdr && n16 < x.E >> 4;
    const bool ok = due.readable && in_pool && sized;
    const uint32_t kind = ok ? (raw ? kDecRaw : kDecPayload) : due.wanted ? kDecZero : kDecSkip;
    r.meta = n16 | (mode << 16) | (kind << 24);
    uint32_t st = 0;
    if (due.stray || (due.wanted && !due.readable)) st = KVC_ST_BAD_INDEX;
    if (due.readable && !ok) st = KVC_ST_CORRUPT;
    if (st) atomicOr(&a.st->status, st);
    return r;
}
template <class P>
__device__ __forceinline__ DecLanes dec_open(const DecodeArgs& a, const DecPlace& t) {
    return dec_check<P>(a, t, dec_ask(a, t));
}

// 16 bytes from global memory straight to LDS: lane l's go to lds + 16 l (the destination is wave-uniform).
// STREAM: and leave what the last-level cache holds where it is (nt).
template <bool STREAM = false>
__device__ __forceinline__ void load_to_lds16(const void* g, void* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g, (__attribute__((address_space(3))) void*)lds, 16, 0, STREAM ? 2 : 0);
}

// Decoder workgroups a compute unit may hold in large calls (0: as many as fit).  With 32 waves on every compute unit,
// 128 KB of 4 KB pages and up to 256 KB of 8 KB pages per compute unit are being written at once, all over the output,
// and the memory serves them worse than 96 to 168 KB.  262,144 pages, decode, us, eight groups -> the number here:
// 16 x 160 335 -> 324, 16 x 192 399 -> 389, 16 x 224 473 -> 459, 16 x 256 541 -> 514; a million of 16 x 128 1009 -> 987, half a
// million of mode 5 502 -> 490 (five groups 1014, seven 1002; 4.5 KB pages 297 -> 301 with six: as many as fit).  The limit is
// LDS that nothing uses.  It holds from 24,576 pages on (16 x 160 30.7 -> 29.6, 16 x 256 45.9 -> 44.7; at 16,384 within half a
// microsecond).  Pages of 6 to 8 KB have one of six groups from 8,192 on, where a call's waves would all be resident at once, or
// nearly, and reach their stores together: 9,216 and 10,240 pages, mode 4, 16 x 192 13.2 -> 12.3 and 14.1 -> 12.8, 13 x 256 13.7 -> 12.8 and
// 14.9 -> 13.8; in cold calls, mode 3, 16 x 192, 8,192 pages 16.7 -> 15.8, 16 x 224, 20,480 36.0 -> 35.0.
// The large calls' limit is for those that decode every block of a range.  Where blocks are named -- id lists, a block table, a prefetch's list of
// blocks to fetch -- many may be left out, and their waves then come and go through fewer places: 131,072 pages in blocks
// of one, three quarters of the ids -1, us, without / with the limit: 16 x 128 44.8 / 57.8, 16 x 256 in blocks of eight 56.2 / 70.3;
// no id -1: 104.3 / 105.8 and 282 / 269; a gather of 655,360 pages that leaves none out 671 / 663.
constexpr int kDecLimitPages = 24576, kDecMiddlePages = 8192;
constexpr int dec_groups(int np, bool partial) { return np == 8 ? 4 : np >= 6 || (np >= 4 && !partial) ? 6 : 0; }
constexpr int dec_groups_middle(int np) { return np >= 6 ? 6 : 0; }
constexpr int kLdsPerCu = 160 * 1024;
// unused LDS per workgroup, beside the kernel's own, that leaves room for `groups` of them
constexpr int dec_spare_lds(int groups, int own) { return groups ? kLdsPerCu / groups - 1280 - own : 0; }  // (1,280: room for the allocation's granularity)

// Whether INT8 payloads go through LDS too.  With several pages per wave their loads have to be under way before
// the first page is stored; with one page per wave they are read straight from the pool, which is 1.5 % faster for
// whole launches of INT8 pages even one pass at a time (262,144 pages of 4 KB: 285 us, 289 us through LDS; more passes
// at a time see below).
template <int PPW>
constexpr bool kStageInt8 = PPW > 1;

// Payloads that are read straight from the pool (INT8 ones with a page per wave, raw ones): how many passes are loaded
// ahead of their stores.  A load waits for the stores before it, so a page takes a trip per step: all passes in one step are 2.4
// us for a call of eight raw pages of 16 x 128, one by one 3.1; and in a transfer engine the one INT8 page of a block is
// what the other fifteen wait for (two steps of 4,370 blocks, of whose pages 6.5 % are INT8: one by one 217 us, all 200).
// A launch of many more pages than the chip holds moves a little faster with less in flight, but a page that dawdles
// keeps its wave from the next: 262,144 INT8 pages of 16 x 128 273 us one by one, 264 by two, 274 all; a million pages of mode 3
// 1008, 996, 997; a gather 686, 666, 666; raw pages 360 one by one, 376 all; INT8 pages of 16 x 256 312 one by one, 280
// all, of 16 x 192 426 and 408, raw ones of 16 x 256 369 and 377.
constexpr int kDecFewPages = 8192;  // 256 compute units of 32 waves
constexpr int dec_int8_step(int np) { return np >= 5 ? np : 2; }

// Start the payload loads of PPW pages, those of lanes first .. first + PPW - 1: the i-th goes to LDS slot i, 16
// bytes per lane and round, without a stop in registers.  Payload bytes past the page's own are not read.
template <class P, int PPW, bool UNIFORM, bool PAST = false>
__device__ __forceinline__ void dec_fetch(const DecodeArgs& a, const DecLanes& L, int first, uint32_t (*slots)[Slot<P::kPasses>::kWords], uint64_t near = ~0ull) {
    const uint32_t lane = (uint32_t)lane_id();
    const bool staged = (L.meta >> 24) == kDecPayload && (kStageInt8<PPW> || ((L.meta >> 16) & 0xFFu) != KVC_MODE_INT8);
    const uint32_t n_own = staged ? L.meta & 0xFFFFu : 0u;
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
        const uint32_t n16 = of_lane<UNIFORM>(n_own, first + i);
        const uint64_t off = of_lane<UNIFORM>(L.off, first + i);
        const uint8_t* src = a.pool + off;
        if (PAST && off >= near) {
#pragma unroll
            for (int z = 0; z < P::kRounds; ++z)
                if (lane + 64u * z < n16) load_to_lds16<true>(src + (lane + 64u * z) * 16u, reinterpret_cast<uint4*>(slots[i]) + 64 * z);
            continue;
        }
#pragma unroll
        for (int z = 0; z < P::kRounds; ++z)
            if (lane + 64u * z < n16) load_to_lds16(src + (lane + 64u * z) * 16u, reinterpret_cast<uint4*>(slots[i]) + 64 * z);
    }
}

// A lane's part of a payload that is read straight from the pool (or, INT8, from its staged copy).
template <bool STREAM>
__device__ __forceinline__ uint2 load_payload(const uint2* p) {
    if constexpr (STREAM) {
        const uint2v v = __builtin_nontemporal_load(reinterpret_cast<const uint2v*>(p));
        return make_uint2(v.x, v.y);
    } else {
        return *p;
    }
}
template <bool STREAM>
__device__ __forceinline__ uint4 load_payload(const uint4* p) {
    if constexpr (STREAM)
        return load_stream(p);
    else
        return *p;
}

// The fetched payloads of this wave are in LDS.  (Waited for before the first output store is issued: loads
// and stores retire in one order, so a payload waited for after a store would wait for the store too.)
__device__ __forceinline__ void dec_fetched() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), the other counters unchanged
    wave_sync();
}

// How the header scan deals packet groups to lanes: pages whose groups divide the wave share a scan.
template <class P>
struct HeaderDeal {
    static constexpr int kG = P::kGroups;
    static constexpr int kSeg = 64 % kG == 0 ? kG : 64;  // lanes per page
    static constexpr int kPages = 64 / kSeg;             // pages per scan
    static constexpr int kRounds = (kG + 63) / 64;       // scans per page
};

// Scan the headers of SCAN <= HeaderDeal<P>::kPages pages, those of slots i0 .. and lanes first + i0 ..: info = what the
// lane's group needs to be read (one per round).  `bad` / `special`: ballots of the lanes whose page fails validation, and of
// the lanes whose group is a zero-run or run packet.
template <class P, bool UNIFORM, int SCAN>
__device__ __forceinline__ void dec_headers(const Extent& x, const DecLanes& L, int first, int i0, const uint32_t (*slots)[Slot<P::kPasses>::kWords],
                                            GroupInfo (&info)[HeaderDeal<P>::kRounds], uint64_t& bad, uint64_t& special) {
    using H = HeaderDeal<P>;
    constexpr int kG = P::kGroups;
    const int lane = lane_id();
    const int pi = i0 + min(lane / H::kSeg, SCAN - 1);  // this lane's page
    const uint32_t meta = SCAN == 1 ? of_lane<UNIFORM>(L.meta, first + i0) : (uint32_t)__builtin_amdgcn_ds_bpermute((first + pi) << 2, (int)L.meta);
    const uint32_t n16 = meta & 0xFFFFu, mode = (meta >> 16) & 0xFFu;
    const uint32_t* stage = SCAN == 1 ? slots[i0] : slots[pi];
    uint32_t total = x.hdr;
    bool wrong = false, rare = false;
#pragma unroll
    for (int r = 0; r < H::kRounds; ++r) {
        const int g = r * 64 + lane % H::kSeg;
        const bool in_page = P::kPartial ? (uint32_t)g < (x.E >> 5) : (kG % H::kSeg == 0 || g < kG);
        // (a group beyond the page: a one-bit literal at the payload's end, read but never stored)
        const uint32_t c = in_page ? (stage[g >> 3] >> ((g & 7) << 2)) & 15u : 1u;
        const uint32_t size = !in_page ? 0u : c == 9 ? 1u : c << 2;
        uint32_t incl;
        if (H::kSeg == 64) {
            incl = wave_incl_scan_dpp(size);
        } else {
            incl = row16_incl_scan_dpp(size);
            if (H::kSeg == 32) incl += dpp<0x142, 0xA>(0, incl);  // odd rows add the row before
        }
        info[r] = group_pack(total + incl - size, c);
        wrong = wrong || c > 9 || (mode == KVC_MODE_DELTA && (c == 0 || c == 9));
        rare = rare || c == 0 || c == 9;
        if (r + 1 < H::kRounds)
            total += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        else
            wrong = wrong || (lane % H::kSeg == H::kSeg - 1 && ((total + incl + 15u) >> 4) != n16);
    }
    const bool packed = (meta >> 24) == kDecPayload && mode != KVC_MODE_INT8;
    bad = __builtin_amdgcn_ballot_w64(packed && wrong);
    special = __builtin_amdgcn_ballot_w64(packed && rare);
}

// Decode an INT8 payload at src (the staged copy, or the pool itself) into the page at dst_b, STEP passes at a time.
template <class P, int STEP, bool STREAM = false>
__device__ __forceinline__ void dec_int8(const DecodeArgs& a, const Extent& x, const LanePos& lp, float s, char* dst_b, const uint2* src) {
    uint2 v[P::kPasses];
#pragma unroll
    for (int p = 0; p < P::kPasses; ++p) {
        if (p % STEP == 0) {
#pragma unroll
            for (int q = p; q < p + STEP && q < P::kPasses; ++q)
                if (lane_live<P>(x, q)) v[q] = load_payload<STREAM>(src + q * 64 + lane_id());
        }
        if (!lane_live<P>(x, p)) continue;
        const uint32_t lo = v[p].x ^ 0x80808080u, hi = v[p].y ^ 0x80808080u;  // + 128 in every byte: the sign bits change
        uint32_t pb[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            pb[k] = lo >> (8 * k);
            pb[4 + k] = hi >> (8 * k);
        }
        store_out(dst_b, pass_base_off<P, false>(a.g, p), pass_lane_off<P, false>(a.g, lp, p), dequant8_biased(pb, s, -128.0f * s));
    }
}

// Copy a raw payload, STEP passes at a time.
template <class P, int STEP, bool STREAM = false>
__device__ __forceinline__ void dec_raw(const DecodeArgs& a, const Extent& x, const LanePos& lp, char* dst_b, const uint4* src) {
    uint4 v[P::kPasses];
#pragma unroll
    for (int p = 0; p < P::kPasses; ++p) {
        if (p % STEP == 0) {
#pragma unroll
            for (int q = p; q < p + STEP && q < P::kPasses; ++q)
                if (lane_live<P>(x, q)) v[q] = load_payload<STREAM>(src + q * 64 + lane_id());
        }
        if (lane_live<P>(x, p)) store_out(dst_b, pass_base_off<P, false>(a.g, p), pass_lane_off<P, false>(a.g, lp, p), v[p]);
    }
}

// Decode one staged packed payload into the page at dst_b.  seg0: the first lane of the page's part of `info`.
// SPECIAL: the page may hold zero-run and run packets.
template <class P, bool SPECIAL>
__device__ __forceinline__ void dec_page(const DecodeArgs& a, const Extent& x, const LanePos& lp, uint32_t mode, float s, char* dst_b, const uint32_t* stage,
                                         const GroupInfo (&info)[HeaderDeal<P>::kRounds], int seg0) {
    constexpr int NP = P::kPasses;
    const int lane = lane_id();
    const float neg128s = -128.0f * s;
    // info of the group this lane's quad unpacks in group set p: lane seg0 + (16 p + quad) mod 64 of its scan
    auto group_info = [&](int p) {
        const uint32_t from = (uint32_t)(seg0 + (p * 16) % 64 + (lane >> 2)) << 2;
        GroupInfo g;
        g.at = (uint32_t)__builtin_amdgcn_ds_bpermute((int)from, (int)info[(p * 16) / 64].at);
        g.high = (uint32_t)__builtin_amdgcn_ds_bpermute((int)from, (int)info[(p * 16) / 64].high);
        return g;
    };
    if constexpr (P::kChan && P::kD == 64) {
        if (mode == KVC_MODE_CHAN) {
            // Mode 5 with eight octets (see the encoder): group set s holds, for this lane, pair 2s + h of its
            // octet over all 16 tokens; the lane's own tokens are values 4h .. 4h + 3 of the packet, the
            // partner's the other four.  The biased codes of a set are kept as bytes, two dwords per set; the
            // lane hands the partner the dword with the partner's tokens and receives the partner's pair for
            // its own tokens.
            const bool hi = lane >= 32;
            uint32_t pair_lo[2], pair_hi[2];  // per set: the dwords of pairs 2s and 2s + 1 for this lane's tokens
#pragma unroll
            for (int sset = 0; sset < 2; ++sset) {
                uint32_t w[2];
                unpack8<NP, SPECIAL>(a, stage, group_info(sset), x.hdr, w);
                const uint32_t own = hi ? w[1] : w[0];  // values 4h .. 4h + 3: this lane's tokens
                const uint32_t got = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)(hi ? w[0] : w[1]));
                pair_lo[sset] = hi ? got : own;  // pair 2s: packed by the lower half's lane
                pair_hi[sset] = hi ? own : got;  // pair 2s + 1: packed by the upper half's lane
            }
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                uint32_t pb[8];
#pragma unroll
                for (int k = 0; k < 8; ++k)  // channel k = pair k / 2 = 2 (k / 4) + (k / 2) % 2, value 2p + k % 2 of the dword
                    pb[k] = (((k >> 1) & 1) ? pair_hi[k >> 2] : pair_lo[k >> 2]) >> (8 * (2 * p + (k & 1)));
                store_out(dst_b, pass_base_off<P, true>(a.g, p), pass_lane_off<P, true>(a.g, lp, p), dequant8_biased(pb, s, neg128s));
            }
            return;
        }
    } else if constexpr (P::kChan) {
        if (mode == KVC_MODE_CHAN) {
            // Mode 5: of a run of 16 octets, group set j holds channels 2j, 2j + 1 of the lane's octet,
            // tokens 4p + (lane & 3) for p = 0..3 (value 2p + e of the packet = pass p, channel 2j + e).  The
            // biased codes of a set are kept as bytes, so that pass p then finds its eight codes at fixed
            // byte positions.
#pragma unroll
            for (int h = 0; h < NP / 4; ++h) {
                uint32_t packed[4][2];
#pragma unroll
                for (int j = 0; j < 4; ++j) unpack8<NP, SPECIAL>(a, stage, group_info(4 * h + j), x.hdr, packed[j]);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    uint32_t pb[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int m = 2 * p + (k & 1);  // value index inside group set k / 2
                        pb[k] = packed[k >> 1][m >> 2] >> (8 * (m & 3));
                    }
                    store_out(dst_b, pass_base_off<P, true>(a.g, 4 * h + p), pass_lane_off<P, true>(a.g, lp, 4 * h + p), dequant8_biased(pb, s, neg128s));
                }
            }
            return;
        }
    }
    const bool no_delta = mode == KVC_MODE_PACK;
    uint32_t carry = 0;  // what a row that continues from the pass before had summed up there
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        uint32_t w[2];
        unpack8<NP, SPECIAL>(a, stage, group_info(p), x.hdr, w);
        uint32_t pb[8];  // codes + 128 in byte 0
        if (no_delta) {  // no delta step was taken: the fields are the codes
#pragma unroll
            for (int k = 0; k < 8; ++k) pb[k] = w[k >> 2] >> (8 * (k & 3));
        } else {
            // prefix sum along the channel index (mod 256): the lanes of the token row before this one, then in the
            // lane.  Every byte carries a bias of 128, so that 128 times the number of bytes summed is in the sum:
            // nothing for a whole lane, and 128 too many at every odd k after adding the 128 of the result.
            const uint32_t t0 = __builtin_amdgcn_udot4(w[0], 0x01010101u, 0u, false);
            const uint32_t tot = __builtin_amdgcn_udot4(w[1], 0x01010101u, t0, false);
            const uint32_t incl = row_incl_scan<P>(lp, p, tot, carry);
            if (!P::kAligned) carry = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            const uint32_t even = incl - tot, odd = even + 128u;
            pb[0] = even + w[0];
            pb[1] = __builtin_amdgcn_udot4(w[0], 0x00000101u, odd, false);
            pb[2] = __builtin_amdgcn_udot4(w[0], 0x00010101u, even, false);
            pb[3] = odd + t0;
            const uint32_t even4 = even + t0;
            pb[4] = even4 + w[1];
            pb[5] = __builtin_amdgcn_udot4(w[1], 0x00000101u, pb[3], false);
            pb[6] = __builtin_amdgcn_udot4(w[1], 0x00010101u, even4, false);
            pb[7] = incl + 128u;
        }
        if (lane_live<P>(x, p))
            store_out(dst_b, pass_base_off<P, false>(a.g, p), pass_lane_off<P, false>(a.g, lp, p), dequant8_biased(pb, s, neg128s));
    }
}

// Decode the pages whose payloads dec_fetch has loaded (dec_fetched: they are there).
template <class P, int PPW, bool UNIFORM, bool PAST = false>
__device__ __forceinline__ void dec_batch(const DecodeArgs& a, const DecLanes& L, int first, const LanePos& lp, uint32_t (*slots)[Slot<P::kPasses>::kWords], bool few,
                                          uint64_t near = ~0ull) {
    using H = HeaderDeal<P>;
    static_assert(PPW % H::kPages == 0 || PPW == 1, "a header scan covers whole pages of the batch");
    constexpr int kScan = PPW < H::kPages ? PPW : H::kPages;  // pages taken from one scan
    const Extent x = page_extent<P>(a.g);
#pragma unroll 1
    for (int i0 = 0; i0 < PPW; i0 += kScan) {
        GroupInfo info[H::kRounds] = {};
        uint64_t bad = 0, special = 0;
        // (a scan for one page is left out where the page has no header: 0.3 us of a small call of INT8 pages)
        const uint32_t meta0 = of_lane<UNIFORM>(L.meta, first + i0);
        if (kScan > 1 || ((meta0 >> 24) == kDecPayload && ((meta0 >> 16) & 0xFFu) != KVC_MODE_INT8))
            dec_headers<P, UNIFORM, kScan>(x, L, first, i0, slots, info, bad, special);
#pragma unroll 1
        for (int j = 0; j < kScan; ++j) {
            const int i = i0 + j;
            const uint32_t meta = of_lane<UNIFORM>(L.meta, first + i);
            const uint32_t kind = meta >> 24;
            if (kind == kDecSkip) continue;
            uint16_t* dst = a.out + page_base(a.g, (int64_t)(int32_t)of_lane<UNIFORM>((uint32_t)L.db, first + i), (int)of_lane<UNIFORM>(L.pg, first + i));
            constexpr uint64_t kSegMask = H::kSeg == 64 ? ~0ull : (1ull << (H::kSeg & 63)) - 1;
            const bool bad_header = ((bad >> (j * H::kSeg)) & kSegMask) != 0;
            if (kind == kDecZero || bad_header) {
                zero_out(dst, a.g);
                if (bad_header && lane_id() == 0) atomicOr(&a.st->status, KVC_ST_CORRUPT);
                continue;
            }
            char* dst_b = reinterpret_cast<char*>(dst);
            if (kind == kDecRaw) {  // stored-uncompressed bypass
                const uint64_t off = of_lane<UNIFORM>(L.off, first + i);
                const uint4* src = reinterpret_cast<const uint4*>(a.pool + off);
                if (PAST && off >= near)
                    dec_raw<P, 1, true>(a, x, lp, dst_b, src);
                else if (few)
                    dec_raw<P, P::kPasses>(a, x, lp, dst_b, src);
                else
                    dec_raw<P, 1>(a, x, lp, dst_b, src);
                continue;
            }
            const uint32_t mode = (meta >> 16) & 0xFFu;
            const float s = __uint_as_float(of_lane<UNIFORM>(__float_as_uint(L.s), first + i));
            if (mode == KVC_MODE_INT8) {
                const uint2* src = kStageInt8<PPW> ? reinterpret_cast<const uint2*>(slots[i]) : reinterpret_cast<const uint2*>(a.pool + of_lane<UNIFORM>(L.off, first + i));
                if (PAST && !kStageInt8<PPW> && of_lane<UNIFORM>(L.off, first + i) >= near)
                    dec_int8<P, dec_int8_step(P::kPasses), true>(a, x, lp, s, dst_b, src);
                else if (kStageInt8<PPW> || few || dec_int8_step(P::kPasses) >= P::kPasses)
                    dec_int8<P, P::kPasses>(a, x, lp, s, dst_b, src);
                else
                    dec_int8<P, dec_int8_step(P::kPasses)>(a, x, lp, s, dst_b, src);
                continue;
            }
            if (((special >> (j * H::kSeg)) & kSegMask) != 0)
                dec_page<P, true>(a, x, lp, mode, s, dst_b, slots[i], info, j * H::kSeg);
            else
                dec_page<P, false>(a, x, lp, mode, s, dst_b, slots[i], info, j * H::kSeg);
        }
    }
}

// PAST: of a call with near_bytes.  (A kernel of its own: asked page by page in the others too, gathers of 51,520 raw pages of 16 x 32 took 18.6
// us, 18.0 without.)
template <class P, bool PAST, int WAVES, int PPW>
__global__ __launch_bounds__(WAVES * 64) void k_decompress(DecodeArgs a) {
    __shared__ __align__(16) uint32_t s_stage[WAVES][PPW][Slot<P::kPasses>::kWords];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t0 = ((int64_t)task_block_index() * WAVES + wave) * PPW;
    // A page's memory chain is ids -> descriptor -> payload, each a full trip to HBM.  The wave walks it for
    // all of its PPW pages at once: lane i resolves page i, then all payload loads are issued, straight to
    // LDS, and the pages are decoded one after the other.
    const LanePos lp = lane_pos<P>(a.g);
    // (a batch of one page is resolved on the scalar unit: every lane has the same task)
    const DecLanes L = dec_open<P>(a, PPW == 1 ? dec_locate(a, t0 < a.n_pages, (uint32_t)t0) : dec_locate(a, lane < PPW && t0 + lane < a.n_pages, (uint32_t)t0 + (uint32_t)lane));
    uint64_t near = ~0ull;
    if constexpr (PAST) {  // (blocks 0, 1, ... of the pool: the first descriptor says where the payloads begin.  Read by the
        near = a.near_bytes;  // scalar unit: a vector load of one line by every wave costs 2 %.)
        if (*(const __attribute__((address_space(4))) uint64_t*)&a.desc[0].off >= near) near = ~0ull;
    }
    dec_fetch<P, PPW, PPW == 1, PAST>(a, L, 0, s_stage[wave], near);
    dec_fetched();
    dec_batch<P, PPW, PPW == 1, PAST>(a, L, 0, lp, s_stage[wave], a.n_pages <= kDecFewPages, near);
}

// Transfer engines of the prefetch window that go turn by turn (Algorithm 1: at most Omega_max transfers outstanding):
// the narrow ones, for calls of many, and wide ones of blocks of few one-pass pages.  A workgroup takes the next issued blocks from the queue (a turn), its waves decode them one block after
// the other, meeting after each -- no payload of a block is asked for before the last store of the engine's block before
// has reached memory --, and the completion is reported before the next turn is taken.  The waves share a block's pages
// as far as they go round (wave w takes pages w, w + WAVES, ...), and queue entries, pool blocks and all descriptors of a
// turn are fetched at once, one page task per lane, before its first payload.  (Looked ahead for as wide engines do it,
// an engine is bound to blocks that an idle one could take: with 546 engines of eight blocks each, on compute units
// that hold two or three, 216 us became 231.)  SIDE: pages of one block that a wave has in flight together.
// (pages of up to four passes whose rows do not cross passes: held within 128 VGPRs, so that four waves fit a SIMD)
template <class P, int WAVES, int SIDE>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(P::kPasses <= 4 && P::kAligned ? 4 : 1))) void k_decompress_window(DecodeArgs a, WindowArgs w) {
    __shared__ __align__(16) uint32_t s_stage[WAVES][SIDE][Slot<P::kPasses>::kWords];
    __shared__ uint32_t s_turn[2];
    __shared__ int32_t s_q[WAVES][2][kMaxWindowTurn];
#if KVC_DEBUG_BOUNDS
    __shared__ uint32_t s_done;  // waves that have finished a block, summed over the engine's blocks
    if (threadIdx.x == 0) s_done = 0;
    uint32_t blocks = 0;  // blocks behind this wave
#endif
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ppb = a.g.ppb;
    const LanePos lp = lane_pos<P>(a.g);
    if (blockIdx.x >= w.hdr->engines) return;  // the window was opened for fewer engines than the grid holds
    // a wave's page tasks of a block, rounded up to whole batches of SIDE pages (tasks past the block do nothing)
    const int per_wave = (ppb + WAVES - 1) / WAVES;
    const int per_block = (per_wave + SIDE - 1) / SIDE * SIDE;
    const uint32_t n_issued = w.hdr->n_issued, chunk = w.hdr->chunk;
    uint32_t mine = 0;
    WindowTurn none;
    none.first = none.count = none.at = 0;
    WindowTurn turn = window_next<true>(w, s_turn, none, s_q[0][0], mine, n_issued, chunk);
    DecLanes L = {};  // 64 page tasks of the turn, one per lane
    int t = 0;        // the wave's page tasks of the turn behind it, in block order
    while (turn.count) {
        if (turn.at == 0) {  // the turn's queue entries and the pool blocks they name, one per lane, parked in the wave's row of LDS
            if ((uint32_t)lane < turn.count) {
                const int32_t slot_l = w.queue[turn.first + lane];
                s_q[wave][0][lane] = slot_l;
                s_q[wave][1][lane] = a.pool_ids[slot_l];
            }
            wave_sync();
            t = 0;
        }
        for (const int end = t + per_block; t < end; t += SIDE) {  // the pages of block number turn.at
            if (t % 64 == 0) {
                const uint32_t b = min((uint32_t)(t + lane) / (uint32_t)per_block, turn.count - 1u);
                DecPlace pl;
                pl.pg = (uint32_t)(wave + (t + lane - (int)b * per_block) * WAVES);
                pl.live = t + lane < (int)turn.count * per_block && (int)pl.pg < ppb;
                pl.bad_index = false;
                pl.pb = s_q[wave][1][b];
                pl.db = s_q[wave][0][b];
                L = dec_open<P>(a, pl);
            }
#if KVC_DEBUG_BOUNDS
            KVC_CHECK(a.st, *(volatile uint32_t*)&s_done >= blocks * WAVES);
#endif
            dec_fetch<P, SIDE, false>(a, L, t % 64, s_stage[wave]);
            dec_fetched();
            dec_batch<P, SIDE, false>(a, L, t % 64, lp, s_stage[wave], true);
            wave_sync();
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the slots have been read before they are filled again
        }
#if KVC_DEBUG_BOUNDS
        if (lane == 0) atomicAdd(&s_done, 1u);
        ++blocks;
#endif
        turn = window_next<false>(w, s_turn, turn, s_q[0][0], mine, n_issued, chunk);
    }
}

// Wide transfer engines of the prefetch window that look ahead, for calls of as many as have a compute unit each, or fewer: a
// workgroup takes issued blocks from the queue in runs, its waves decode them one block after the other,
// meeting after each -- no payload of a block is asked for before the last store of the engine's block before has
// reached memory.  An engine is latency, not bandwidth: few of them are at work, each on one block.  So the waves share a
// block's pages as far as they go round (there is one for each of 16), and what leads to a payload -- ticket, queue entry,
// pool block, descriptors, four trips one after the other -- is walked ahead of the payloads by one of the waves, the clerk,
// a trip per block: while the payloads of block i are on their
// way it asks for the descriptors of block i + 1 (a page per lane), the pool block of i + 2, the queue entry of i + 3 and,
// where its run ends, the next run; while block i is decoded it publishes block i + 1 and keeps the books.  Two steps of
// 4,370 blocks of 16 pages of 16 x 128, us, 256 / 16 engines: 230 / 2,090 with the trips walked for a run at a time, when the
// run before had ended; 238 / 2,342 looked ahead for by every wave (a few hundred instructions in 16 waves); 217 / 2,017 by
// a clerk; and of its last form, with INT8 pages loaded ahead, 200 / 2,009 when it published between the barriers and
// 196 / 1,909 now.
// (pages of up to four passes whose rows do not cross passes: held within 128 VGPRs, so that four waves fit a SIMD)
template <class P, int WAVES>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(P::kPasses <= 4 && P::kAligned ? 4 : 1))) void k_decompress_window_wide(WindowParams params) {
    const DecodeArgs& a = params.a;
    constexpr int kClerkPages = 64;  // pages of a block the clerk looks up; blocks of more are left to the waves
    constexpr int kClerk = WAVES - 1;
    __shared__ __align__(16) uint32_t s_stage[WAVES][1][Slot<P::kPasses>::kWords];
    __shared__ __align__(16) uint4 s_page[kClerkPages];  // the block at work: what the waves need to know of its pages,
    __shared__ int32_t s_block[2];                       // its slot (-1: there is none) and its pool block
    __shared__ WindowBooks s_books;                      // the clerk's (in LDS, not in registers of all waves)
#if KVC_DEBUG_BOUNDS
    __shared__ uint32_t s_done;  // waves that have finished a block, summed over the engine's blocks
    if (threadIdx.x == 0) s_done = 0;
    uint32_t behind = 0;  // meetings behind this wave
#endif
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool clerk = wave == kClerk;
    const int ppb = a.g.ppb;
    const LanePos lp = lane_pos<P>(a.g);
    const uint32_t engines = params.w.hdr->engines, n_issued = params.w.hdr->n_issued, chunk = params.w.hdr->chunk;
    if (blockIdx.x >= engines) return;  // the window was opened for fewer engines than the grid holds
    const int per_block = (ppb + WAVES - 1) / WAVES;  // a wave's page tasks of a block (tasks past the block do nothing)
    const bool looked_up = ppb <= kClerkPages;
    auto page_task = [&](bool live, int pg, int32_t slot, int32_t pb) {
        DecPlace pl;
        pl.pg = (uint32_t)pg;
        pl.live = live && pg < ppb;
        pl.bad_index = false;
        pl.pb = pb;
        pl.db = slot;
        return pl;
    };

    auto clerk_task = [&](int32_t slot, int32_t pb) { return page_task(looked_up && slot >= 0, lane, slot, pb); };
    // the clerk: what the waves are to do next
    auto publish = [&](const DecLanes& pages, int32_t next_slot, int32_t next_pb) {
        s_page[lane] = make_uint4((uint32_t)pages.off, (uint32_t)(pages.off >> 32), __float_as_uint(pages.s), pages.meta);
        if (lane == 0) {
            s_block[0] = next_slot;
            s_block[1] = next_pb;
        }
    };
    if (clerk) {
        __builtin_amdgcn_s_setprio(3);  // whatever it does beside its pages, the others wait for (217 us, without 229)
        const WindowParams& k = params_again<WindowParams>();
        WindowBooks b;
        b.open_at(n_issued, blockIdx.x, engines, chunk);
        // the first three entries, one per lane: a trip for all queue entries and one for all pool blocks
        const uint32_t i0 = b.take(), i1 = b.take(), i2 = b.take();  // (engines <= n_issued: there is a first)
        const uint32_t i = lane == 0 ? i0 : lane == 1 ? i1 : lane == 2 ? i2 : kWindowNone;
        int32_t slot_i = -1, pb_i = -1;
        if (i != kWindowNone) slot_i = k.w.queue[i];
        if (slot_i >= 0) pb_i = k.a.pool_ids[slot_i];
        const int32_t slot0 = __builtin_amdgcn_readlane(slot_i, 0), pb0 = __builtin_amdgcn_readlane(pb_i, 0);
        b.slot1 = __builtin_amdgcn_readlane(slot_i, 1);
        b.slot2 = __builtin_amdgcn_readlane(slot_i, 2);
        b.pb1 = __builtin_amdgcn_readlane(pb_i, 1);
        b.layer = b.layer_of(k.w, slot0);
        b.put(s_books);
        publish(dec_open<P>(k.a, clerk_task(slot0, pb0)), slot0, pb0);
    }
    // The loop and its exit branch on the scalar unit, and the single-wave and single-lane parts lie in the middle of its
    // body: every wave meets every barrier with all of its lanes.  (With single-lane work at both ends of the loop body the
    // compiler merges it across the back edge into an outer loop and lets the other lanes run ahead to the next barrier:
    // the workgroup then never meets.)  Of the two barriers per block the first says that the clerk has published
    // the next block (and that the block before has been read), the second that all stores of this one are in memory.
    int32_t slot = -1, pb = -1;
    DecLanes L;
    // page tasks t .. t + 63 of the block, one per lane
    auto lanes = [&](int t) {
        const int pg = wave + (t + lane) * WAVES;
        if (!looked_up) return dec_open<P>(params_again<WindowParams>().a, page_task(t + lane < per_block, pg, slot, pb));
        const uint4 v = s_page[min(pg, kClerkPages - 1)];
        DecLanes r;
        r.off = (uint64_t)v.x | ((uint64_t)v.y << 32);
        r.s = __uint_as_float(v.z);
        r.meta = pg < ppb && slot >= 0 ? v.w : 0u;
        r.pg = (uint32_t)pg;
        r.db = slot;
        return r;
    };
    auto meet = [&]() {
        __syncthreads();
        slot = wave_uniform(s_block[0]);
        pb = wave_uniform(s_block[1]);
        L = lanes(0);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), the other counters unchanged
#if KVC_DEBUG_BOUNDS
        if (lane == 0) atomicAdd(&s_done, 1u);
#endif
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
    };
    meet();
    while (slot >= 0) {
#if KVC_DEBUG_BOUNDS
        ++behind;
#endif
        for (int t = 0;;) {
#if KVC_DEBUG_BOUNDS
            KVC_CHECK(a.st, *(volatile uint32_t*)&s_done >= behind * WAVES);
#endif
            dec_fetch<P, 1, false>(a, L, t % 64, s_stage[wave]);
            if (t == 0 && clerk) {
                const WindowParams& k = params_again<WindowParams>();
                WindowBooks b;
                b.get(s_books);
                const uint4 asked = dec_ask(k.a, clerk_task(b.slot1, b.pb1));
                int32_t pb2 = b.slot2 < 0 ? -1 : k.a.pool_ids[b.slot2];
                const uint32_t i3 = b.take();
                int32_t slot3 = i3 == kWindowNone ? -1 : k.w.queue[i3];
                const uint32_t run = b.next_run();
                uint32_t ticket = 0;
                if (lane == 0) {
                    if (run) ticket = atomicAdd(&k.w.hdr->ticket, run);
                    if (b.rep) {
                        const long long now = max(wall_clock64(), 1ll);  // read before the blocks are counted
                        if (atomicSub(&k.w.pending[b.rep_layer], (int)b.rep) == (int)b.rep) window_stamp(&k.w.notify[k.w.layer_begin + (int32_t)b.rep_layer], now);
                    }
                }
                if (run) b.refill((uint32_t)wave_uniform((int32_t)ticket), run);
                publish(dec_check<P>(k.a, clerk_task(b.slot1, b.pb1), asked), b.slot1, b.pb1);
                b.block_done(k.w);
                b.slot1 = b.slot2;
                b.slot2 = wave_uniform(slot3);
                b.pb1 = wave_uniform(pb2);
                b.put(s_books);
            }
            dec_fetched();
            dec_batch<P, 1, false>(a, L, t % 64, lp, s_stage[wave], true);
            wave_sync();
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the slots have been read before they are filled again
            if (++t >= per_block) break;
            if (t % 64 == 0) L = lanes(t);
        }
        meet();
    }
    if (clerk && lane == 0) {
        const WindowArgs& w = params_again<WindowParams>().w;
        const WindowBooks& b = s_books;
        if (b.rep && atomicSub(&w.pending[b.rep_layer], (int)b.rep) == (int)b.rep) window_stamp(&w.notify[w.layer_begin + (int32_t)b.rep_layer], max(wall_clock64(), 1ll));
        window_leave(w, b.mine, w.hdr->n_issued);
    }
}

// Launch shapes by page size (NP passes of 1 KB): waves per workgroup, pages per wave.
constexpr int kCodecWaves = 4;
// Transfer engines of the prefetch window.  Calls of at most as many engines (omega, or the slots of the call) as the
// device holds of the wide kind -- one per compute unit, 256, at 16 x 128; two where the kernel fits 64 vector registers --
// have engines of 16 waves; the others have engines of four waves, with several pages of a block per wave in flight, of
// which four to seven fit a compute unit.  Two prefetch steps of 2,048 blocks of 16 pages of 16 x 128, us, four-wave
// engines / wide engines that fetched a run at a time, all else alike: 64 engines 498 / 320, 256 engines 160 / 121; blocks of
// two pages, where most waves of a wide engine have none, 735 / 748 with 64 engines (wide engines have gained a sixth
// to a quarter since).  (The choice is made before the transfers are counted: an omega above the wide kind's number with few
// transfers runs 256 narrow engines; and as wide engines are now, more engines than the device holds of them can be
// slower than as many as it does: 4,370 blocks of 16 pages of 16 x 128 a step, two steps, omega 256 / 512 / 1,024 180 / 198 / 187 us.)
constexpr int kWideWaves = 16;
// Wide engines of blocks of up to this many one-pass pages go turn by turn like narrow ones.  Such a block is decoded
// sooner than its clerk has walked ahead, and with a page for every wave the clerk's own comes on top.  Two steps of 20 layers x
// 64 sequences x 8 blocks, us, with a clerk / turn by turn: 16 x 32, 8 engines, blocks of 1 page 3,155 / 2,745, 4 3,527 / 3,490, 8
// 3,596 / 3,694, 16 4,709 / 4,104, 24 (8 layers) 2,180 / 2,313; 256 engines 137 / 116, 150 / 144, 154 / 153, 186 / 169, 112 / 121;
// 7 x 32 in blocks of 16 4,657 / 3,787 and 184 / 155; 16 x 64 in blocks of 16, 32 engines 666 / 723.
constexpr int kTurnPages = 16;
constexpr int window_side(int np) { return np <= 4 ? 4 : 2; }
// Pages per decoder wave: a page of one or two passes is too small to cover its own memory chain, so a wave
// takes the pages that share a header scan, resolved one per lane.  Measured (half a million pages, us): one
// pass 180 / 112 / 117 with 1 / 4 / 8 pages, two passes 283 / 276 / 294 with 1 / 2 / 4, four passes 1075 / 1083 /
// 1109 (a million pages) with 1 / 2 / 4: there the launch moves 5.8 TB/s, what a copy does, with any of them.
constexpr int dec_ppw(int np) { return np == 1 ? 4 : np == 2 ? 2 : 1; }
// ... unless the call is small: then the memory chain is walked once anyway, and pages side by side are decoded sooner than
// one after the other (16 x 64, us, two pages per wave -> one: 8 pages 6.4 -> 6.0, 1,024 6.8 -> 6.0, 8,192 9.1 -> 8.8,
// 16,384 12.3 -> 12.5; 16 x 32, four -> one: 1,024 6.9 -> 6.0, 4,096 7.2 -> 6.3, 16,384 9.3 -> 10.8).
constexpr int kDecSmallPages(int np) { return 4096 * np; }

// Encoder launch shapes of calls below the large ones: workgroups of `waves` waves with `ppw` pages each, up to `pages`
// pages.  Such a call (a decode step's offload, a sequence's) is latency: one page per wave while the cursor bears it.
// It serves an atomic per workgroup every 13 ns, so the more pages there are, the more have to share one -- first by
// more waves in the workgroup, then by more pages per wave, which follow one another.  The lines lie where a shape stops
// being resident at once (16 waves of one page: 4,096 pages, 8,192 where the kernel fits 64 registers; 8 of four pages: 16,384):
// beyond its line it is slower than what comes next.  Compress with a cursor reset before it, us, workgroups of four
// waves of 1 (up to 2,048) and of 4 or 5 pages -> these, 16 x 128: 1,024 pages 13.8 -> 12.9, 2,048 17.1 -> 14.5, 4,096
// 18.9 -> 17.0, 8,192 22.9 -> 19.9, 16,384 31.8 -> 28.2 (12,288 with eight waves of four 26.3, four of four 25.2); 16 x 64, two
// pages per wave -> these: 8 11.3 -> 10.5, 1,024 12.3 -> 11.8, 4,096 16.2 -> 14.5, 16,384 21.3 -> 20.0; 16 x 32, four ->
// these: 8 11.7 -> 9.9, 1,024 12.3 -> 11.4, 4,096 15.8 -> 13.2, 16,384 19.3 -> 18.7; 16 x 256: 1,024 15.8 -> 15.0, 4,096
// 21.9 -> 20.9; a mode per block: 16 x 96 4,096 24.1 -> 15.4, 16 x 64 8,192 25.3 -> 18.2, 16 x 128 4,096 22.6 -> 17.7
// (beyond that the waves of 16 are no longer resident at once: 5,120 to 8,192 pages 5 to 14 % faster in cold calls with modes that
// change from block to block, but 7 to 18 % slower with modes that don't and with blocks of one page).
struct EncTier {
    int pages, waves, ppw;
};
constexpr int kEncTiers = 5;
constexpr EncTier enc_tier(int np, int scheme, int i) {
    constexpr EncTier none = {0, 4, 1};
    constexpr EncTier one[kEncTiers] = {{512, 4, 1}, {1024, 8, 1}, {16384, 16, 2}, {32768, 16, 4}, none};  // one pass
    constexpr EncTier two[kEncTiers] = {{512, 4, 1}, {2048, 8, 1}, {16384, 16, 2}, none, none};
    constexpr EncTier three[kEncTiers] = {{512, 4, 1}, {1024, 8, 1}, {8192, 16, 1}, none, none};
    constexpr EncTier any_four[kEncTiers] = {{512, 4, 1}, {1024, 8, 1}, {4096, 16, 1}, none, none};  // four, the mode read at run time
    constexpr EncTier four[kEncTiers] = {{512, 4, 1}, {1024, 8, 1}, {8192, 16, 1}, {13312, 4, 4}, {16384, 8, 4}};
    constexpr EncTier pairs[kEncTiers] = {{512, 4, 1}, {1024, 8, 1}, {4096, 16, 1}, {13312, 4, 4}, {32768, 8, 4}};  // four, mode 5
    constexpr EncTier six[kEncTiers] = {{512, 4, 1}, {3072, 8, 1}, none, none, none};                          // five and six
    constexpr EncTier more[kEncTiers] = {{512, 4, 1}, {4096, 8, 1}, none, none, none};
    return np == 1 ? one[i] : np == 2 ? two[i] : np == 3 ? three[i] : np == 4 ? (scheme < 0 ? any_four[i] : scheme == KVC_MODE_CHAN ? pairs[i] : four[i]) : np <= 6 ? six[i] : more[i];
}
// Where the mode is read at run time but is the same for all blocks, the large shapes are reached earlier: the pages of a
// workgroup are then done together, and plain INT8 and raw ones soon (16 x 128, 4,096 INT8 pages 14.7 us against 15.8; 16 x 32,
// 16,384 INT8 pages 16.7 against 18.0).
constexpr int enc_uniform_pages(int np, int scheme) {
    const bool plain = scheme == KVC_MODE_RAW || scheme == KVC_MODE_INT8;
    return plain ? (np <= 2 ? 8192 : 2048) : 1 << 30;
}

inline dim3 page_grid(int64_t n_pages, int ppw, int waves = kCodecWaves) {
    const int64_t per_wg = (int64_t)waves * ppw;
    return dim3((unsigned)((n_pages + per_wg - 1) / per_wg));
}

// The host side of one page shape: picks the instantiation and launches it.
template <int D, int NP, bool PARTIAL>
struct ShapeOps {
    using P = Page<D, NP, PARTIAL>;

    template <int SCHEME, int TIER>
    static bool compress_tier(const EncodeArgs& a, hipStream_t s, hipError_t& r) {
        constexpr EncTier t = enc_tier(NP, SCHEME, TIER);
        if constexpr (t.pages > 0) {
            if (a.n_pages <= t.pages) {
                r = launch_kernel(k_compress<P, t.waves, t.ppw, SCHEME>, page_grid(a.n_pages, t.ppw, t.waves), dim3(t.waves * 64), s, a);
                return true;
            }
        }
        return false;
    }

    template <int SCHEME>
    static hipError_t compress_scheme(const EncodeArgs& a, hipStream_t s) {
        hipError_t r = hipSuccess;
        if (SCHEME < 0 && a.block_scheme == nullptr && a.n_pages > enc_uniform_pages(NP, a.scheme)) {
            // large
        } else if (compress_tier<SCHEME, 0>(a, s, r) || compress_tier<SCHEME, 1>(a, s, r) || compress_tier<SCHEME, 2>(a, s, r) || compress_tier<SCHEME, 3>(a, s, r) || compress_tier<SCHEME, 4>(a, s, r)) {
            return r;
        }
        constexpr EncShape e = enc_large(NP, SCHEME);
        return launch_kernel(k_compress<P, e.waves, e.ppw, SCHEME>, page_grid(a.n_pages, e.ppw, e.waves), dim3(e.waves * 64), s, a);
    }

    static hipError_t compress(const EncodeArgs& a, hipStream_t s) {
        // the full scheme of Algorithm 2 for every block is the common launch and gets its own
        // instantiation; any other request (another mode, or one mode per block) reads it at run time,
        // and so do all requests for pages with a short last pass
        if constexpr (PARTIAL) {
            return a.scheme == KVC_MODE_CHAN ? hipErrorInvalidValue : compress_scheme<kSchemeRowMajor>(a, s);
        } else {
            if (a.block_scheme == nullptr && a.scheme == KVC_MODE_RLE) return compress_scheme<KVC_MODE_RLE>(a, s);
            if (a.block_scheme == nullptr && a.scheme == KVC_MODE_CHAN) {
                // channel-pair groups: its own instantiations (another deal of the page to the lanes)
                if constexpr (P::kChan)
                    return compress_scheme<KVC_MODE_CHAN>(a, s);
                else
                    return hipErrorInvalidValue;
            }
            // one mode per block: where the shape has mode 5, the instantiation that can also deal a page by channel pairs
            if constexpr (P::kChan) {
                if (a.block_scheme != nullptr) return compress_scheme<kSchemeAny>(a, s);
            }
            return compress_scheme<kSchemeRowMajor>(a, s);
        }
    }

    static hipError_t decompress(const DecodeArgs& a, hipStream_t s) {
        if constexpr (dec_ppw(NP) > 1) {
            if (a.n_pages <= kDecSmallPages(NP)) return launch_kernel(k_decompress<P, false, kCodecWaves, 1>, page_grid(a.n_pages, 1), dim3(kCodecWaves * 64), s, a);
        }
        constexpr int own = kCodecWaves * dec_ppw(NP) * Slot<NP>::kBytes, groups = dec_groups(NP, PARTIAL), middle = dec_groups_middle(NP);
        constexpr int spare = dec_spare_lds(groups, own), spare_middle = dec_spare_lds(middle, own);
        static_assert(spare >= 0 && (groups == 0 || own + spare > kLdsPerCu / (groups + 1)), "one group more does not fit");
        static_assert(spare_middle >= 0 && (middle == 0 || own + spare_middle > kLdsPerCu / (middle + 1)), "one group more does not fit");
        const bool whole = !a.pool_ids && !a.dst_ids && !a.block_table;
        const int lds = a.n_pages < kDecMiddlePages ? 0 : a.n_pages < kDecLimitPages ? spare_middle : whole ? spare : 0;
        const auto kernel = a.near_bytes != ~0ull ? k_decompress<P, true, kCodecWaves, dec_ppw(NP)> : k_decompress<P, false, kCodecWaves, dec_ppw(NP)>;
        return launch_kernel_lds(kernel, page_grid(a.n_pages, dec_ppw(NP)), dim3(kCodecWaves * 64), lds, s, a);
    }

    // whether the wide engines of blocks of ppb pages are of the kind that looks ahead
    static bool window_looks_ahead(int ppb) { return NP > 1 || ppb > kTurnPages; }

    static hipError_t decompress_window(const DecodeArgs& a, const WindowArgs& w, unsigned grid, bool wide, hipStream_t s) {
        if constexpr (NP == 1) {
            if (wide && !window_looks_ahead(a.g.ppb)) return launch_kernel(k_decompress_window<P, kWideWaves, 1>, dim3(grid), dim3(kWideWaves * 64), s, a, w);
        }
        if (wide) return launch_kernel(k_decompress_window_wide<P, kWideWaves>, dim3(grid), dim3(kWideWaves * 64), s, WindowParams{a, w});
        return launch_kernel(k_decompress_window<P, kCodecWaves, window_side(NP)>, dim3(grid), dim3(kCodecWaves * 64), s, a, w);
    }

    // engines the current device holds at once: a larger grid would only queue workgroups behind the
    // resident ones, which keep taking turns until the queue is empty
    static int window_capacity(bool wide, int ppb) {
        int dev = 0, cus = 0, per_cu = 0;
        const void* k = wide ? reinterpret_cast<const void*>(&k_decompress_window_wide<P, kWideWaves>) : reinterpret_cast<const void*>(&k_decompress_window<P, kCodecWaves, window_side(NP)>);
        if constexpr (NP == 1) {
            if (wide && !window_looks_ahead(ppb)) k = reinterpret_cast<const void*>(&k_decompress_window<P, kWideWaves, 1>);
        }
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, (wide ? kWideWaves : kCodecWaves) * 64, 0) != hipSuccess) {
            (void)hipGetLastError();
            return 0;  // unknown: no cap (narrow), never used (wide)
        }
        return cus * per_cu;
    }

    static constexpr ShapeKernels kTable = {D, NP, PARTIAL, &compress, &decompress, &decompress_window, &window_capacity, &window_looks_ahead};
};

}  // namespace
}  // namespace kvc
