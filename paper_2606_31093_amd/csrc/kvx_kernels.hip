// kvx_kernels.hip -- the copy engine of libkvx: HIP kernels for gfx950.
//
// They move the rows named by a batch of request records from a
// source side to a destination side (Omni-Flow Sec. 4.1.1: layer x page x
// slice addressing; Sec. 4.1.2: conversion between the paged layout and the
// flat serialization; Sec. 5.2: slot -> page translation through a table).
// Nothing is computed on the data: every element moves as raw bytes inside
// 16-byte vectors, so the kernels are bound by HBM (or the host link when a
// side is pinned host memory).
//
// The unit of work is one page of the tiling side in one layer; the tiling
// side is the destination pool for transfer and
// scatter (each unit then writes one destination page of one layer, and no
// two units write the same bytes) and the source pool for gather.  Three
// kernels share the work out:
// - kvx_sweep_kernel: a planned transfer, one workgroup of one wavefront per
//   kilobyte of a unit, started in order by the hardware;
// - kvx_order_kernel: unplanned calls of long records whose tokens are runs
//   on both sides, a persistent grid that keeps that order;
// - kvx_parts_kernel (kvx_shared_parts_kernel for more than 64 records): the
//   other unplanned calls (few or short records, rows to resolve, the host
//   link), a persistent grid over parts of units.
//
// Order matters because of the memory, not of the caches: nothing is re-read.
// A bare copy of random 256 KiB pages moves 6.6 TB/s (read + write) when the
// kilobytes in flight all lie in a few pages being walked through, and 5.1 to
// 6.3 TB/s, depending on where the pools sit in physical memory, when every
// wavefront walks through a page of its own.

#include <algorithm>
#include <atomic>

#include "kvx_internal.h"

#ifndef KVX_NT
#define KVX_NT 1   // streaming (non-temporal) loads and stores: nothing is re-read
#endif
#ifndef KVX_NT_LOAD
#define KVX_NT_LOAD KVX_NT
#endif
#ifndef KVX_NT_STORE
#define KVX_NT_STORE KVX_NT
#endif
// kvx_parts_kernel: workgroups of 256 threads per CU, and 16-byte vectors in
// flight per lane (64 decode records, 1-4 tokens of 36 x 8 x 128: 12.2 us).
#ifndef KVX_PARTS_BLOCKS_PER_CU
#define KVX_PARTS_BLOCKS_PER_CU 7
#endif
#ifndef KVX_PARTS_UNROLL
#define KVX_PARTS_UNROLL 4
#endif
// kvx_shared_parts_kernel: threads per workgroup, which share their look at the
// records, and workgroups per CU; where rows are resolved, workgroups of 256
// threads.  16384 records of 1-4 tokens of 2 x 2 x 64, and 4096 of 36 x 8 x 128:
// 512 threads, 3 per CU, 100 and 638 us; 1024, 1, 70 and 685; 256, 7, 169 and 635.
#ifndef KVX_SHARE_BLOCK
#define KVX_SHARE_BLOCK 512
#endif
#ifndef KVX_SHARE_BLOCKS_PER_CU
#define KVX_SHARE_BLOCKS_PER_CU 3
#endif
#ifndef KVX_SHARE_ROWS_BLOCKS_PER_CU
#define KVX_SHARE_ROWS_BLOCKS_PER_CU 6
#endif
// Parts per wavefront that units are cut into.  64 half-filled pages of 36
// layers: 111 us with 16 to 64.
#ifndef KVX_GRID_PARTS
#define KVX_GRID_PARTS 32
#endif
// Unplanned calls that resolve rows: from KVX_TEAM_KIB KiB per wavefront of the
// grid on, in units that most often hold KVX_TEAM_UNIT vectors or belong to records
// of many pages, four wavefronts share a part, and of the grid only
// KVX_TEAM_BLOCKS_PER_CU workgroups per CU work, KVX_TEAM_PARTS parts per wavefront.
// A wavefront to itself walks through a page of its own, and thousands of pages at
// once run at the memory's random rate.  Teams, head-major 64 to token-major 64 token pages, 100 records of 400
// to 800 tokens of 36 x 8 x 128: 2 per CU 3249 us, 3 3311, 4 3319; the way
// back 3026, 3155 and 3197.  Calls of less data lie in the last-level cache, read and
// written, and have more parts than teams without them: 4 records of 130 tokens, 153
// MB, 36.3 us in teams, 30.6 without; 16 of 48, 226 MB, 47.4 and 44.5; 32 of 32, 302 MB,
// 59.5 and 60.7; 48 of 40, 566 MB, 105.8 and 112.  Small units fill no
// team, unless they are small pages of long records (KVX_TEAM_PAGES or more of them):
// 2000 records of 1 to 8 tokens, 4 heads of 256 bytes 376 us in teams, 268 without;
// 24-token pages of 3 x 80 bytes, 2.0 GB, 490 and 534.
#ifndef KVX_TEAM_KIB
#define KVX_TEAM_KIB 32
#endif
#ifndef KVX_TEAM_UNIT
#define KVX_TEAM_UNIT 4096
#endif
#ifndef KVX_TEAM_PAGES
#define KVX_TEAM_PAGES 4
#endif
#ifndef KVX_TEAM_PARTS
#define KVX_TEAM_PARTS 1
#endif
#ifndef KVX_TEAM_BLOCKS_PER_CU
#define KVX_TEAM_BLOCKS_PER_CU 2
#endif
// The same over the host link: 8 vectors per lane (4: 1.8% slower), and units
// cut into as many parts as make KVX_LINK_PARTS of the call: fewer do not fill
// the link, and many units in parts are slower.  Out and back, 1 page of 2
// layers: 27 us, 242 in whole units; 2 x 8 layers 163 (80 parts 165, 320 168,
// 640 183, whole units 333); 8 x 36 layers 2688 (2684, 2701, 2726, 2692).
#ifndef KVX_LINK_BLOCKS_PER_CU
#define KVX_LINK_BLOCKS_PER_CU 5
#endif
#ifndef KVX_LINK_PARTS
#define KVX_LINK_PARTS 160
#endif
#ifndef KVX_LINK_UNROLL
#define KVX_LINK_UNROLL 8
#endif
// kvx_order_kernel: threads per workgroup, one workgroup per CU (256 KiB
// pages, 43.7 GB: 7.0-7.35 ms; 512 threads, two workgroups, 7.05-7.2 ms, but
// 72 KiB pages 5.1 against 4.75 ms and 288 KiB serializations 2.43 against
// 2.28 ms).
#ifndef KVX_ORDER_BLOCK
#define KVX_ORDER_BLOCK 1024
#endif
// Which calls keep the order, judged on the device by the first 64 records:
// full pages of at least KVX_ORDER_PIECES KiB, three quarters filled,
// KVX_ORDER_TURNS KiB to copy per wavefront, and pages of the other side that
// begin between pieces.  Below them there is no order to keep: 1-4 tokens of 64
// records 18.3 us in order, 12.2 in parts; half-filled pages 126 us in order, 112
// in parts.  Order against parts, 32 long prompts and 8 of them (us): 40 KiB
// pages 4410 : 4347, 217 : 211; 48 KiB 4355 : 4384, 214 : 211; 52 KiB 4366 : 4413,
// 316 : 326; 56 KiB 4256 : 4404, 315 : 332; 64 KiB 3712 : 4378, 177 : 201; 256 KiB
// 7245 : 8690.  Where a page of the other side begins inside a piece that piece
// resolves its rows, and at the barrier all wait for it: MLA's 72 KiB pages from
// a shifted start 6308 : 4183, 96 KiB of 3 x 80 from one 2208 : 1824.  Where units
// are taken in turns, all pieces of a unit in several such pages do (64 to 128
// token pages of 1 x 576, 7.4 GB: 1892 : 1519).
#ifndef KVX_ORDER_PIECES
#define KVX_ORDER_PIECES 52
#endif
#ifndef KVX_ORDER_QUARTERS
#define KVX_ORDER_QUARTERS 3
#endif
#ifndef KVX_ORDER_TURNS
#define KVX_ORDER_TURNS 16
#endif
// ... and, on the host, calls whose table holds this many entries per record: a
// small call with a table longer than its records need takes 14.2 us in
// workgroups of 1024 threads, 12.2 without (64 decode records).
#ifndef KVX_ORDER_PAGES
#define KVX_ORDER_PAGES 8
#endif

namespace kvx {
namespace {

constexpr int kBlock = 256;   // threads of a parts workgroup
constexpr int kWave = 64;
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4u ld16(const char *p) {
#if KVX_NT_LOAD
    return __builtin_nontemporal_load(reinterpret_cast<const v4u *>(p));
#else
    return *reinterpret_cast<const v4u *>(p);
#endif
}

// Stores into device memory stream past the caches; stores into pinned host
// memory (HOST) are ordinary, which measured faster over PCIe.
template <bool HOST>
__device__ __forceinline__ void st16(char *p, v4u v) {
#if KVX_NT_STORE
    if (!HOST) {
        __builtin_nontemporal_store(v, reinterpret_cast<v4u *>(p));
        return;
    }
#endif
    *reinterpret_cast<v4u *>(p) = v;
}

// A read of data the kernel never writes (the plan, the records, the page
// tables) through the constant address space: the compiler may then serve a
// uniform one from the scalar cache wherever it falls, also after stores.
template <class T>
__device__ __forceinline__ T cload(const T *ptr) {
    static_assert(sizeof(T) % 4 == 0, "whole 32-bit words");
    typedef const __attribute__((address_space(4))) uint32_t cword;
    const cword *q = (const cword *)(uintptr_t)ptr;
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = q[i];
    T out;
    __builtin_memcpy(&out, w, sizeof(T));
    return out;
}

__device__ __forceinline__ void report(const Params &p, uint32_t bits) {
    if (p.err) atomicOr(p.err, bits);
}

// A record as the plan's check sees it.
struct Req {
    int64_t t_pt_off, o_pt_off;  // table offsets of the destination / source
    int64_t pages;               // destination pages it touches
    int32_t t_start, o_start, n;
    int32_t j0;                  // first destination page (logical)
};

__device__ __forceinline__ bool load_req(const Params &p, int32_t r, Req &q) {
    const kvx_req &R = p.reqs[r];
    q.t_pt_off = R.dst_pt_off;
    q.o_pt_off = R.src_pt_off;
    q.t_start = R.dst_start;
    q.o_start = R.src_start;
    q.n = R.n_tokens;
    q.j0 = 0;
    q.pages = 0;
    if (q.n < 0 || q.o_start < 0 || q.t_start < 0 || R.reserved != 0 ||
        (int64_t)q.o_start + q.n > INT32_MAX || (int64_t)q.t_start + q.n > INT32_MAX)
        return false;
    if (q.n == 0) return true;
    q.j0 = (int32_t)fd_div(p.fd_Tt, (uint32_t)q.t_start);
    q.pages = (int32_t)fd_div(p.fd_Tt, (uint32_t)(q.t_start + q.n - 1)) - q.j0 + 1;
    return true;
}

// Lane k's row of a sweep piece: kv component c, slot, head h, vector v of
// the row, in the vector order of a unit (TOKENS: token by token; else, for
// a head-major destination, in blocks of KVX_SWEEP_SLOT_BLOCK slots); valid is
// cleared for a masked slot of a head-major destination.
template <bool TOKENS>
__device__ __forceinline__ void tile_row(uint32_t H, uint32_t vpr, const FastDiv &fd_H,
                                         const FastDiv &fd_vpr, uint32_t k, uint32_t rows_c, int32_t sa,
                                         int32_t sb, uint32_t blk0, uint32_t &c, uint32_t &slot,
                                         uint32_t &h, uint32_t &v, bool &valid) {
    constexpr uint32_t SB = KVX_SWEEP_SLOT_BLOCK;
    const uint32_t rw = fd_div(fd_vpr, k);
    v = k - rw * vpr;
    c = rw >= rows_c;
    const uint32_t rr = rw - c * rows_c;
    if (TOKENS) {
        const uint32_t tt = fd_div(fd_H, rr);
        h = rr - tt * H;
        slot = (uint32_t)sa + tt;
    } else {
        const uint32_t q1 = rr / SB;
        const uint32_t blk = fd_div(fd_H, q1);
        h = q1 - blk * H;
        slot = (blk0 + blk) * SB + (rr - q1 * SB);
        valid = valid && slot >= (uint32_t)sa && slot < (uint32_t)sb;
    }
}

// What the copying part of the sweep reads of its arguments.
struct SweepArgs {
    const kvx_plan_slot *slots;
    FastDiv ppt;                 // pieces per page slot
    FastDiv pages;               // page slots per layer: the plan's pages
    uint32_t slot0, n_slots;     // page slots of this launch: [slot0, slot0 + n_slots) of layers x pages
    uint32_t checks;             // leading workgroups that check the plan (a multiple of 8)
    uint32_t general;            // nonzero: strides too large for the fields below
    const int32_t *d_pt, *s_pt;
    uint32_t d_last, s_last;     // last index of each page table
    uint32_t d_T, s_T, d_lastp, s_lastp;   // slots per page, last page id
    FastDiv fd_To;
    FastDiv fd_hv;               // vectors of one token's copied heads
    uint32_t C;
    uint32_t d_t, s_t;           // bytes from one slot to the next
    uint32_t d_c, s_c;           // bytes from K to V
    uint32_t d_l, d_p, s_l, s_p; // 16-byte units from one layer or page to the next
    char *d_base;
    const char *s_base;
    uint32_t H, vpr, d_h, s_h;   // rows only
    FastDiv fd_H, fd_vpr;        // rows only
};

// How a piece's vectors lie on both sides:
// - RUNS: the copied heads of consecutive tokens are one run on both sides;
// - TOKENS: the copied heads of a token are one run on both sides;
// - ROWS_T: token by token into a token-major destination, rows resolved;
// - ROWS_H: by slot blocks into a head-major destination, rows resolved (the
//   sweep takes a head range of a token-major destination the same way).
enum SweepMode { RUNS, TOKENS, ROWS_T, ROWS_H };

// A piece that the sweep's common path does not cover: rows in several source
// pages, a page id or index out of range, or strides too large for 32-bit
// fields.  Every lane resolves its own source page, and errors are
// reported for the positions the piece covers, destination first.
template <bool TOKEN_ORDER, bool HOST>
__device__ __forceinline__ void sweep_piece_general(const Params &p, const kvx_plan_slot &d, uint32_t l,
                                                    uint32_t kb) {
    const Side &ts = p.dst, &os = p.src;
    const int32_t sa = d.dst_slot, so_a = d.src_slot;
    const uint32_t ntok = (uint32_t)d.n_tokens;
    const int32_t sb = sa + (int32_t)ntok;
    constexpr uint32_t SB = KVX_SWEEP_SLOT_BLOCK;
    const uint32_t blk0 = (uint32_t)sa / SB, nblk = ((uint32_t)sb - 1) / SB - blk0 + 1;
    const uint32_t rows_c = TOKEN_ORDER ? ntok * p.H : p.H * nblk * SB;
    const uint32_t total = rows_c * p.vpr * (uint32_t)p.C;
    const uint32_t k = kb + threadIdx.x;
    bool valid = k < total;
    uint32_t c, slot, h, v;
    tile_row<TOKEN_ORDER>(p.H, p.vpr, p.fd_H, p.fd_vpr, valid ? k : total - 1, rows_c, sa, sb, blk0, c, slot,
                          h, v, valid);
    if (!valid) return;
    // Tables hold at most INT32_MAX entries, so 32-bit unsigned compares also
    // reject negative indices.
    const bool t_in = (uint32_t)d.dst_idx < (uint32_t)ts.pt_len;
    const int32_t tpage = t_in ? cload(ts.pt + (uint32_t)d.dst_idx) : -1;
    if ((uint32_t)tpage >= (uint32_t)ts.N) {
        report(p, t_in ? KVX_DERR_DST_PAGE : KVX_DERR_PT_RANGE);
        return;
    }
    const uint32_t pos = (uint32_t)so_a + (slot - (uint32_t)sa);
    const uint32_t jo = fd_div(p.fd_To, pos);
    const int64_t idx = (int64_t)d.src_idx + jo;
    if (idx < 0 || idx >= os.pt_len) {
        report(p, KVX_DERR_PT_RANGE);
        return;
    }
    const int32_t pg = os.pt[idx];
    if (pg < 0 || pg >= os.N) {
        report(p, KVX_DERR_SRC_PAGE);
        return;
    }
    const uint32_t so = pos - jo * (uint32_t)os.T;
    const char *src = os.base + (int64_t)l * os.s_l + (int64_t)pg * os.s_p + c * os.s_c + (int64_t)so * os.s_t +
                      (int64_t)h * os.s_h + v * 16;
    char *dst = ts.base + (int64_t)l * ts.s_l + (int64_t)tpage * ts.s_p + c * ts.s_c + (int64_t)slot * ts.s_t +
                (int64_t)h * ts.s_h + v * 16;
    st16<HOST>(dst, ld16(src));
}

// One piece of the sweep: the vectors [kb, kb + 64) of page slot d of layer
// l, one per lane, in the vector order of its mode.  The common path, a piece
// whose rows lie in one source page with every index and page id in range,
// needs the two page ids and nothing else, read through the scalar cache;
// returns false for any other piece, before anything was copied or reported.
// d's slots are in range already.  Indices are clamped into the tables, so
// that the page ids can be on their way while the checks are made.
template <SweepMode MODE, bool HOST>
__device__ __forceinline__ bool sweep_piece(const SweepArgs &a, const kvx_plan_slot &d, uint32_t l,
                                            uint32_t kb) {
    constexpr bool kRows = MODE == ROWS_T || MODE == ROWS_H;
    constexpr uint32_t SB = KVX_SWEEP_SLOT_BLOCK;
    const uint32_t sa = (uint32_t)d.dst_slot, so_a = (uint32_t)d.src_slot, ntok = (uint32_t)d.n_tokens;
    const uint32_t blk0 = sa / SB, nblk = (sa + ntok - 1) / SB - blk0 + 1;
    const uint32_t rows_c = MODE == ROWS_H ? a.H * nblk * SB : ntok * a.H;
    const uint32_t R = kRows ? rows_c * a.vpr : ntok * a.fd_hv.d;      // vectors per kv component
    const uint32_t total = R * a.C;
    const uint32_t kk = kb + threadIdx.x, k = kk < total ? kk : total - 1;
    uint32_t od, os, jo0 = 0, bad = a.general;
    bool valid = kk < total;
    if (!kRows) {
        if (so_a + ntok > a.s_T) {
            // the source pages of the piece's first and last token
            const uint32_t ke = (kb + kWave < total ? kb + kWave : total) - 1;
            const bool c0 = kb >= R, c1 = ke >= R;
            uint32_t t0 = fd_div(a.fd_hv, c0 ? kb - R : kb), t1 = fd_div(a.fd_hv, c1 ? ke - R : ke);
            if (c0 != c1) t0 = 0, t1 = ntok - 1;
            jo0 = fd_div(a.fd_To, so_a + t0);
            bad |= fd_div(a.fd_To, so_a + t1) - jo0;
        }
    } else {
        uint32_t c, slot, h, v;
        tile_row<MODE == ROWS_T>(a.H, a.vpr, a.fd_H, a.fd_vpr, k, rows_c, sa, sa + ntok, blk0, c, slot, h, v,
                                 valid);
        const uint32_t jo = fd_div(a.fd_To, so_a + (slot - sa));
        const uint64_t live = __ballot(valid);
        if (live == 0) return true;
        jo0 = __builtin_amdgcn_readlane(jo, __builtin_ctzll(live));
        bad |= __ballot(valid && jo != jo0) != 0;
        od = (c ? a.d_c : 0) + (slot - sa) * a.d_t + h * a.d_h + v * 16;
        os = (c ? a.s_c : 0) + (slot - sa) * a.s_t + h * a.s_h + v * 16;
    }
    const uint32_t didx = (uint32_t)d.dst_idx, sidx = (uint32_t)d.src_idx + jo0;
    const uint32_t di = didx < a.d_last ? didx : a.d_last, si = sidx < a.s_last ? sidx : a.s_last;
    const uint32_t dpage = (uint32_t)cload(a.d_pt + di), spage = (uint32_t)cload(a.s_pt + si);
    // (jo0 < 2^21 cannot carry a non-negative src_idx past 2^32)
    bad |= (didx ^ di) | (sidx ^ si) | ((uint32_t)d.src_idx >> 31);
    const uint32_t dp = dpage < a.d_lastp ? dpage : a.d_lastp, sp = spage < a.s_lastp ? spage : a.s_lastp;
    bad |= (dpage ^ dp) | (spage ^ sp);
    if (bad) return false;
    char *dd = a.d_base + (((uint64_t)l * a.d_l + (uint64_t)dp * a.d_p) << 4) + (uint64_t)sa * a.d_t;
    // the source slot of the page's first token, counted from source page jo0
    const char *ss = a.s_base + (((uint64_t)l * a.s_l + (uint64_t)sp * a.s_p) << 4) +
                     (int64_t)((int32_t)so_a - (int32_t)(jo0 * a.s_T)) * a.s_t;
    if (!kRows) {
        // (lanes past the last vector repeat it)
        const bool c = k >= R;
        const uint32_t w = c ? k - R : k, t = MODE == TOKENS ? fd_div(a.fd_hv, w) : 0;
        od = w * 16 + (c ? a.d_c : 0) + t * (a.d_t - a.fd_hv.d * 16);
        os = w * 16 + (c ? a.s_c : 0) + t * (a.s_t - a.fd_hv.d * 16);
        st16<HOST>(dd + od, ld16(ss + os));
    } else if (valid) {
        st16<HOST>(dd + od, ld16(ss + os));
    }
    return true;
}

__device__ __forceinline__ int32_t clamp_i32(int64_t x) {
    return x < INT32_MIN ? INT32_MIN : x > INT32_MAX ? INT32_MAX : (int32_t)x;
}

// Whether slot d of the plan is page qi of the plan the records imply: its
// record's prefix range holds qi, and its fields are those of that record's
// page qi - prefix[r].
__device__ __forceinline__ bool slot_agrees(const Params &p, int64_t qi, const kvx_plan_slot &d) {
    const int32_t r = d.req;
    if (r < 0 || r >= p.n_reqs) return false;
    Req q;
    if (!load_req(p, r, q)) return false;
    const int64_t jj = qi - p.prefix[r];
    if (jj < 0 || qi >= p.prefix[r + 1] || jj >= q.pages) return false;
    const int64_t j = (int64_t)q.j0 + jj, page_lo = j * p.dst.T;
    const int64_t q_end = (int64_t)q.t_start + q.n;
    const int64_t qa = page_lo > q.t_start ? page_lo : q.t_start;
    const int64_t qb = page_lo + p.dst.T < q_end ? page_lo + p.dst.T : q_end;
    const int64_t pos = qa - q.t_start + q.o_start;
    const int64_t jo = pos / p.src.T;
    return d.dst_idx == clamp_i32(q.t_pt_off + j) && d.src_idx == clamp_i32(q.o_pt_off + jo) &&
           d.dst_slot == (int32_t)(qa - page_lo) && d.n_tokens == (int32_t)(qb - qa) &&
           d.src_slot == (int32_t)(pos - jo * p.src.T);
}

// The checking workgroups of a sweep (`n` of them): the plan's slots against
// the records, a lane per slot; prefix[0] = 0, prefix[r + 1] - prefix[r] =
// pages of record r, and prefix[n_reqs] = plan_pages.  Malformed records are
// reported too.
__device__ __forceinline__ void sweep_check(const Params &p, uint32_t b, uint32_t n) {
    const int64_t first = (int64_t)b * kWave + threadIdx.x, step = (int64_t)n * kWave;
    bool bad_plan = first == 0 && (p.prefix[0] != 0 || p.prefix[p.n_reqs] != p.plan_pages);
    for (int64_t qi = first; qi < p.plan_pages; qi += step)
        bad_plan = bad_plan || !slot_agrees(p, qi, p.slots[qi]);
    for (int64_t r = first; r < p.n_reqs; r += step) {
        Req mine;
        if (!load_req(p, (int32_t)r, mine)) report(p, KVX_DERR_BAD_REQ);
        bad_plan = bad_plan || p.prefix[r + 1] - p.prefix[r] != mine.pages;
    }
    if (bad_plan) report(p, KVX_DERR_BAD_PLAN);
}

// Sweep kernel (a planned pool -> pool transfer): one wavefront per
// workgroup, and workgroup b copies one piece of 64 vectors (1 KiB) of one
// destination page of one layer, found by one read of the
// plan.  Workgroups are numbered layer by layer and page slot by page slot
// within a layer (pages in plan order), so the hardware dispatcher, which
// starts them in order, keeps the pieces in flight on the whole GPU inside a
// small window that slides through the transfer.  The dispatcher
// deals consecutive workgroups to the 8 XCDs in turn, so within each group
// of 8 page slots the numbering gives XCD x every piece of slot x, in order:
// each page is copied by one XCD (1.5-6% more than pieces dealt across XCDs).
// What bounds it: a wavefront's life before its load.  With 32 wavefronts per
// CU, 1 KiB each is what the memory wants in flight (a bare copy in this order
// moves 6.6-6.7 TB/s; 2 KiB per wavefront 6.2-6.4, whole pages per wavefront
// 5.1), so every cycle spent on finding the piece is rate lost.  Hence three
// waits (arguments, plan slot, page ids), indices clamped instead of branched
// on, the plan's check in workgroups of its own, and all that is rare in
// sweep_piece_general.  Measured on 256 KiB pages (36 x 8 x 128, 43.7 GB):
// 7129 us with the checks and the rare paths inline, three passes over the
// pages; 6613 us so.  72 KiB pages (61 x 576): 4371 to 4238 us; head ranges in
// 4-layer launches of 300 MB: 499 to 460 us.
// SPARSE: a page has a workgroup per piece of its average part (a.ppt), and
// pages that hold more are copied in turns.  Empty pieces would cost a third to
// two thirds of copied ones: 256 pages of 256 KiB, 16 of 64 tokens each, in
// 4-layer launches, 542 us with a workgroup per piece of the whole page, 271 so.
// Full pages lose 1.2% by the loop, so they have no use for it.
template <SweepMode MODE, bool HOST, bool SPARSE>
__global__ void __launch_bounds__(kWave) kvx_sweep_kernel(SweepArgs a, Params) {
    // The second argument is read where it is needed: a piece on the common
    // path needs nothing of it, and its fields would crowd the scalar
    // registers.
    typedef const __attribute__((address_space(4))) char *ConstPtr;
    ConstPtr args = (ConstPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const Params &p = *(const Params *)(args + sizeof(SweepArgs));
    // The first is read at once, with one wait.
    asm volatile("" ::"s"(a.slots), "s"(a.ppt.d), "s"(a.ppt.m), "s"(a.ppt.l), "s"(a.pages.d), "s"(a.pages.m),
                 "s"(a.pages.l), "s"(a.slot0), "s"(a.n_slots), "s"(a.checks), "s"(a.general), "s"(a.d_pt),
                 "s"(a.s_pt), "s"(a.d_last), "s"(a.s_last), "s"(a.d_T), "s"(a.s_T), "s"(a.d_lastp),
                 "s"(a.s_lastp));
    asm volatile("" ::"s"(a.fd_hv.d), "s"(a.C), "s"(a.d_t), "s"(a.s_t), "s"(a.d_c), "s"(a.s_c), "s"(a.d_l),
                 "s"(a.d_p), "s"(a.s_l), "s"(a.s_p), "s"(a.d_base), "s"(a.s_base));
    uint32_t b = blockIdx.x;
    if (b < a.checks) {
        sweep_check(p, b, a.checks);
        return;
    }
    b -= a.checks;
    // In each whole group of 8 page slots, XCD b % 8 takes slot 8g + b % 8
    // (its pieces in order); the last slots, fewer than 8, one after the other.
    const uint32_t g = fd_div(a.ppt, b >> 3);
    uint32_t slot = (g << 3) + (b & 7u), part = (b >> 3) - g * a.ppt.d;
    if ((g << 3) + 8u > a.n_slots) {
        const uint32_t r = b - (g << 3) * a.ppt.d, s = fd_div(a.ppt, r);
        slot = (g << 3) + s;
        part = r - s * a.ppt.d;
    }
    slot += a.slot0;
    const uint32_t l = fd_div(a.pages, slot);
    kvx_plan_slot d = cload(a.slots + (slot - l * a.pages.d));
    asm volatile("" ::"s"(d.dst_idx), "s"(d.src_slot));   // the whole slot with one wait
    // The slot is trusted only as far as keeping every access inside the
    // pools and tables; whether it matches the records is checked separately.
    const uint32_t sa = (uint32_t)d.dst_slot < a.d_T - 1 ? (uint32_t)d.dst_slot : a.d_T - 1;
    const uint32_t ntok = (uint32_t)d.n_tokens < a.d_T - sa ? (uint32_t)d.n_tokens : a.d_T - sa;
    const uint32_t so_a = (uint32_t)d.src_slot < a.s_T - 1 ? (uint32_t)d.src_slot : a.s_T - 1;
    d.dst_slot = (int32_t)sa;
    d.n_tokens = (int32_t)ntok;
    d.src_slot = (int32_t)so_a;
    constexpr uint32_t SB = KVX_SWEEP_SLOT_BLOCK;
    const uint32_t slots = MODE == ROWS_H && ntok ? ((sa + ntok - 1) / SB - sa / SB + 1) * SB : ntok;
    const uint32_t vecs = slots * a.fd_hv.d * a.C;
    uint32_t kb = part * kWave;
    if (kb >= vecs) return;
    do {
        if (!sweep_piece<MODE, HOST>(a, d, l, kb)) sweep_piece_general<MODE != ROWS_H, HOST>(p, d, l, kb);
        kb += a.ppt.d * kWave;
    } while (SPARSE && kb < vecs);
}

// What the persistent grid reads of its arguments.  `t` is the tiling side,
// `o` the other one; strides inside a page are in 16-byte vectors, which fit
// 32 bits (a page of one layer has fewer than 2^31).
struct GridArgs {
    const kvx_req *reqs;
    uint32_t *err;
    int32_t n_reqs;
    char *t_base, *o_base;
    int64_t t_l, t_p, o_l, o_p;       // bytes from one layer or page to the next
    const int32_t *t_pt, *o_pt;
    int64_t t_len, o_len;
    int64_t cap_bytes;                // buffer side
    int64_t token_bytes;              // one token of a buffer's block
    uint32_t t_N, o_N;
    uint32_t C, elem_shift;
    uint32_t t_c, t_t, o_c, o_t;
    FastDiv fd_Tt, fd_To, fd_hv, fd_L;
    uint32_t granule;                 // tokens after which a whole number of 64 vectors ends; 0: full units in turns
    uint32_t t_h, o_h;                // rows only
    uint32_t slot_shift;              // ROWS_H: log2 of the slots per block
    FastDiv fd_vpr, fd_H;             // rows only
    uint64_t team_min;                // rows only: vectors from which teams of wavefronts share a part,
    uint32_t team_blocks;             // and the workgroups that then work
    float even, team_even;            // part size aimed at, in 64 U (256 U for teams) vectors, for each 64 vectors
                                      // of a wavefront's 64 records
};

// A record as the grid sees it: the part of it whose tiling-side pages the
// table holds.
struct GridRec {
    int64_t t_idx;     // table index of its first tiling-side page
    int64_t o_off;     // table offset (pool) or byte offset (buffer) of the other side
    int64_t pages;     // its tiling-side pages; 0: nothing to copy
    int32_t sa;        // slot of its first token
    int32_t n;         // tokens
    int32_t pos;       // other-side position of its first token
    int32_t n_block;   // tokens of its block (buffer side)
};

// Works out record R (g.pages is 0 when there is nothing to copy); returns
// the error bits it raises.  Every field is computed whatever the record
// holds, without a branch.
template <int OP>
__device__ __forceinline__ uint32_t grid_record(const GridArgs &a, const kvx_req &R, GridRec &g) {
    const int64_t so = R.src_pt_off, dof = R.dst_pt_off, bo = R.buf_off;
    const int32_t s0 = R.src_start, d0 = R.dst_start, n = R.n_tokens;
    bool ok = n >= 0 && s0 >= 0 && d0 >= 0 && R.reserved == 0 && (int64_t)s0 + n <= INT32_MAX &&
              (int64_t)d0 + n <= INT32_MAX;
    if (OP != OP_TRANSFER) {
        const int64_t most = a.cap_bytes >> a.elem_shift, at = (bo < 0 ? 0 : bo > most ? most : bo) << a.elem_shift;
        ok = ok && (OP == OP_GATHER ? d0 : s0) == 0 && bo >= 0 && bo <= most && (at & 15) == 0 &&
             at + (int64_t)n * a.token_bytes <= a.cap_bytes;
    }
    const int64_t T = a.fd_Tt.d;
    const int64_t t_off = OP == OP_GATHER ? so : dof;
    const int64_t t_start = OP == OP_GATHER ? s0 : d0, o_start = OP == OP_GATHER ? d0 : s0;
    const uint32_t first = ok ? (uint32_t)t_start : 0, last = ok && n > 0 ? (uint32_t)(t_start + n - 1) : 0;
    // tiling-side pages [j0, j1], and of those the ones the table holds (a
    // table offset beyond the 2^31 pages of a record either way holds none)
    const int64_t j0 = fd_div(a.fd_Tt, first), j1 = fd_div(a.fd_Tt, last);
    const int64_t far = (int64_t)1 << 32;
    const int64_t off = t_off < -far ? -far : t_off > a.t_len ? a.t_len : t_off;
    const int64_t lo = off < 0 ? -off : 0, hi = a.t_len - 1 - off;
    const int64_t k0 = j0 > lo ? j0 : lo, k1 = j1 < hi ? j1 : hi;
    const int64_t from = j0 < lo ? lo * T : t_start, to = j1 > hi ? (hi + 1) * T : t_start + n;
    const bool some = ok && n > 0;
    g.t_idx = off + k0;
    g.o_off = OP == OP_TRANSFER ? so : (int64_t)((uint64_t)bo << a.elem_shift);
    g.pages = some && k0 <= k1 ? k1 - k0 + 1 : 0;
    g.sa = (int32_t)(from - k0 * T);
    g.n = (int32_t)(to - from);
    g.pos = (int32_t)(from - t_start + o_start);
    g.n_block = n;
    return !ok ? KVX_DERR_BAD_REQ : some && (k0 != j0 || k1 != j1) ? KVX_DERR_PT_RANGE : 0;
}

// Inclusive sum over the wavefront's lanes, without LDS.
__device__ __forceinline__ uint64_t wave_scan(uint64_t x) {
#define KVX_DPP_ADD(ctrl, rows)                                                                            \
    {                                                                                                      \
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, ctrl, rows, 0xf, false);      \
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), ctrl, rows, 0xf, false); \
        x += ((uint64_t)hi << 32) | lo;                                                                    \
    }
    KVX_DPP_ADD(0x111, 0xf)   // row_shr 1, 2, 4, 8: the 16 lanes of a row
    KVX_DPP_ADD(0x112, 0xf)
    KVX_DPP_ADD(0x114, 0xf)
    KVX_DPP_ADD(0x118, 0xf)
    KVX_DPP_ADD(0x142, 0xa)   // row_bcast 15 into rows 1 and 3
    KVX_DPP_ADD(0x143, 0xc)   // row_bcast 31 into rows 2 and 3
#undef KVX_DPP_ADD
    return x;
}

__device__ __forceinline__ uint32_t wave_scan32(uint32_t x) {
#define KVX_DPP_ADD(ctrl, rows) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, false);
    KVX_DPP_ADD(0x111, 0xf)   // the same steps
    KVX_DPP_ADD(0x112, 0xf)
    KVX_DPP_ADD(0x114, 0xf)
    KVX_DPP_ADD(0x118, 0xf)
    KVX_DPP_ADD(0x142, 0xa)
    KVX_DPP_ADD(0x143, 0xc)
#undef KVX_DPP_ADD
    return x;
}

// Largest of the lanes' values, in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_xor((int)x, d, kWave);
        x = x > y ? x : y;
    }
    return x;
}

__device__ __forceinline__ uint32_t lane32(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ int64_t lane64(int64_t v, int lane) {
    return ((int64_t)lane32((uint32_t)(v >> 32), lane) << 32) | lane32((uint32_t)v, lane);
}

// A part of a unit (a page of a layer): the vectors [kb, ke) of its K run and
// then its V run, or of its tokens' runs.
struct GridPart {
    char *t;             // tiling side at the unit's first token, K
    const char *o;       // other side there (ONE), or its layer
    uint64_t o_c;        // other side: bytes from K to V
    int64_t o_off;
    uint32_t kb, ke;
    uint32_t R;          // vectors of one kv component
    uint32_t pos;        // other-side position of the first token
    uint32_t sa, ntok;   // ROWS_H: slot of the first token, tokens
};

// Slots that a unit's vectors enumerate: its tokens, or (ROWS_H) the whole
// blocks of 1 << sb slots that they meet.
template <SweepMode MODE>
__device__ __forceinline__ uint32_t unit_slots(uint32_t sa, uint32_t ntok, uint32_t sb) {
    return MODE == ROWS_H ? (((sa + ntok - 1) >> sb) - (sa >> sb) + 1) << sb : ntok;
}

// The most of them that a page of a record has.
template <SweepMode MODE>
__device__ __forceinline__ uint32_t record_slots(const GridRec &g, uint32_t T, uint32_t sb) {
    if (g.pages == 0) return 0;
    const uint32_t n = (uint32_t)g.n < T ? (uint32_t)g.n : T;
    if (MODE != ROWS_H) return n;
    const uint32_t some = ((n - 1) >> sb) + 2, all = ((T - 1) >> sb) + 1;
    return (some < all ? some : all) << sb;
}

// Token (from the unit's first one; out of range for a masked slot), head and
// vector of the row of vector w of a kv component.
template <SweepMode MODE>
__device__ __forceinline__ void unit_row(const GridArgs &a, uint32_t sa, uint32_t w, uint32_t &tok, uint32_t &h,
                                         uint32_t &v) {
    if (MODE == ROWS_H) {
        const uint32_t sb = a.slot_shift, rw = fd_div(a.fd_vpr, w), q1 = rw >> sb, blk = fd_div(a.fd_H, q1);
        v = w - rw * a.fd_vpr.d;
        h = q1 - blk * a.fd_H.d;
        tok = (((sa >> sb) + blk) << sb) + (rw - (q1 << sb)) - sa;
    } else {
        tok = fd_div(a.fd_hv, w);
        v = w - tok * a.fd_hv.d;
        h = 0;
        if (MODE == ROWS_T) {
            h = fd_div(a.fd_vpr, v);
            v -= h * a.fd_vpr.d;
        }
    }
}

// Vector kk of a part: where it is read and written; false for none.  ONE:
// the part's tokens lie in one page of the other side (always for a buffer),
// which g.o points into; else page_of(jo) gives the id of the other side's
// logical page jo (~0: none).
template <int OP, SweepMode MODE, bool ONE, class PageOf>
__device__ __forceinline__ bool part_vector(const GridArgs &a, const GridPart &g, uint32_t kk, PageOf page_of,
                                            const char *&src, char *&dst) {
    const uint32_t k = kk < g.ke ? kk : g.ke - 1;
    bool valid = kk < g.ke;
    const bool c = k >= g.R;
    const uint32_t w = c ? k - g.R : k;     // vector of the kv component
    uint32_t to = w, oo = w;                // offsets in vectors
    const char *ol = g.o;
    if (MODE != RUNS || !ONE) {
        uint32_t tok, h, v;
        unit_row<MODE>(a, g.sa, w, tok, h, v);
        if (MODE == ROWS_H) valid = valid && tok < g.ntok;
        to = tok * a.t_t + v;
        oo = ONE ? tok * a.o_t + v : v;
        if (MODE == ROWS_T || MODE == ROWS_H) {
            to += h * a.t_h;
            oo += h * a.o_h;
        }
        if (!ONE) {
            const uint32_t q = g.pos + tok, jo = fd_div(a.fd_To, q), pg = page_of(jo, valid);
            valid = valid && pg != ~0u;
            ol += (int64_t)pg * a.o_p + (uint64_t)(q - jo * a.fd_To.d) * a.o_t * 16;
        }
    }
    char *tp = g.t + ((uint64_t)to + (c ? a.t_c : 0)) * 16;
    const char *op = ol + (uint64_t)oo * 16 + (c ? g.o_c : 0);
    src = OP == OP_GATHER ? tp : op;
    dst = OP == OP_GATHER ? const_cast<char *>(op) : tp;
    return valid;
}

// Copies a part, U vectors per lane in flight: thread `me` of the `span` that
// share it.  Lanes without a vector load one all the same, that of the part's
// last or the source's first: between loads that some lanes skip the compiler
// waits for all that is in flight, which left one or two of the U (200 tokens of
// 36 x 8 x 128 with a padded table 18.8 us so, 15.5 with all four in flight;
// gathered from 16 records of 1 to 20 tokens and scattered 35.5 and 30.2).
template <int OP, SweepMode MODE, bool ONE, bool HOST, int U, class PageOf>
__device__ __forceinline__ void copy_part(const GridArgs &a, const GridPart &g, uint32_t me, uint32_t span,
                                          PageOf page_of) {
    for (uint32_t k0 = g.kb; k0 < g.ke; k0 += span * U) {            // the same trip count for every lane
        const char *src[U];
        char *dst[U];
        bool have[U];
        v4u val[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            have[u] = part_vector<OP, MODE, ONE>(a, g, k0 + u * span + me, page_of, src[u], dst[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            val[u] = ld16(have[u] || (ONE && MODE != ROWS_H) ? src[u] : OP == OP_GATHER ? a.t_base : a.o_base);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (have[u]) st16<HOST>(dst[u], val[u]);
    }
}

// The id of the other side's page `idx` of its table, ~0 (and reported) when
// there is none.
__device__ __forceinline__ uint32_t other_page(const GridArgs &a, int64_t idx) {
    const bool in = idx >= 0 && idx < a.o_len;
    const uint32_t pg = in ? (uint32_t)a.o_pt[idx] : ~0u;
    if (pg < a.o_N) return pg;
    if (a.err) atomicOr(a.err, in ? KVX_DERR_SRC_PAGE : KVX_DERR_PT_RANGE);
    return ~0u;
}

__device__ __forceinline__ kvx_req load_raw(const GridArgs &a, int32_t r) {
    kvx_req R{};
    if (r < a.n_reqs) R = a.reqs[r];
    return R;
}

// The arguments, read anew: kept over all of a kernel they would not fit the
// scalar registers.
__device__ __forceinline__ const GridArgs &fresh_args() {
    typedef const __attribute__((address_space(4))) GridArgs *ConstArgs;
    ConstArgs ap = (ConstArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    return *(const GridArgs *)ap;
}

// The records of a workgroup of B threads that share their look at them.
template <int B>
struct Records {
    GridRec rec[B];
    int64_t end[B];              // parts up to and with record i's, among its 64
    uint32_t parts[B];           // parts of each of record i's pages
    uint32_t part_vecs[B];       // vectors of each part
};

// Whether four wavefronts share each part, judged by 64 of the records, one per
// lane (`chunks` times as many in all), whose largest pages hold `tile` vectors.
__device__ __forceinline__ bool worth_teams(const GridArgs &a, const GridRec &g, uint32_t tile, uint32_t chunks) {
    const uint64_t some = __ballot(g.pages > 0), large = __ballot(
        g.pages > 0 && (tile >= KVX_TEAM_UNIT || (g.pages >= KVX_TEAM_PAGES && tile >= 4 * kWave)));
    const uint64_t all = (uint64_t)lane64(wave_scan((uint64_t)g.pages * tile), kWave - 1) * a.fd_L.d * chunks;
    return all >= a.team_min && 2 * __builtin_popcountll(large) >= __builtin_popcountll(some);
}

// Persistent grid over parts of units, for calls of few or short records and
// for those that resolve rows.
// Every wavefront looks at 64 records, one per lane: a scan over the lanes
// turns their parts into ranges, and the record of a part is found with one
// ballot and read with lane reads.  A call of up to 64 records needs no LDS
// and no barrier: every wavefront looks at all of them.  Of more, each
// wavefront of a workgroup looks at another 64 and leaves what it found in
// LDS: looking at 64 records costs a wavefront about 0.5 us whether or not
// any of their parts are its own (1024, 16384 and 65536 records of 1-4 tokens of
// 2 x 2 x 64: 36, 533 and 2119 us when every wavefront looked at all of them, 7.8,
// 100 and 387 so).
// What bounds a small call is the chain of dependent
// loads (records, page ids of both sides at once, data) and the width of the
// chip: a unit is cut into parts of 64 U vectors, or larger ones once there
// are KVX_GRID_PARTS per wavefront.  Layers are innermost, so that the parts
// in flight spread over the pool.  Against whole units per wavefront and
// records in LDS (us, that : this): 64 decode records 14.4 : 12.2, 64
// half-filled pages 145 : 112, 4 x 50 tokens 38.9 : 15.2, 1024 decode records
// 162 : 157, 16384 of them 2494 : 2504.
template <int OP, SweepMode MODE, bool HOST, int U, int B, bool SHARE>
__device__ __forceinline__ void copy_parts(Records<B> *shared) {
    constexpr bool kPool = OP == OP_TRANSFER, kRows = MODE == ROWS_T || MODE == ROWS_H;
    constexpr uint32_t kUnit = kWave * U, kTeam = 4;
    constexpr int kWaves = B / kWave, kStep = SHARE ? B : kWave;
    const uint32_t lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t n_reqs = fresh_args().n_reqs;
    uint32_t team = 1, me = lane, workers = gridDim.x * kWaves;
    int64_t at = (int64_t)blockIdx.x * kWaves + wave;
    if (SHARE && kRows) {
        const GridArgs &a = fresh_args();
        GridRec g;
        (void)grid_record<OP>(a, load_raw(a, lane), g);
        const uint32_t tile = record_slots<MODE>(g, a.fd_Tt.d, a.slot_shift) * a.fd_hv.d * a.C;
        if (worth_teams(a, g, tile, (n_reqs + kWave - 1) / kWave)) {
            if (blockIdx.x >= a.team_blocks) return;
            workers = a.team_blocks * kWaves;
            team = kTeam;
            me = threadIdx.x % (kTeam * kWave);
            at /= kTeam;
        }
    }
    for (int32_t r0 = 0; r0 < (SHARE ? n_reqs : 1); r0 += kStep) {
        const GridArgs &ra = fresh_args();
        const uint32_t L = ra.fd_L.d, T = ra.fd_Tt.d;
        GridRec g;                                         // (a lane without a record has an empty one)
        const uint32_t bad = grid_record<OP>(ra, load_raw(ra, r0 + (SHARE ? threadIdx.x : lane)), g);
        if (bad && blockIdx.x == 0 && (SHARE || wave == 0) && ra.err) atomicOr(ra.err, bad);
        const uint32_t tile = record_slots<MODE>(g, T, ra.slot_shift) * ra.fd_hv.d * ra.C;   // vectors of the record's largest page
        if (!SHARE && kRows && worth_teams(ra, g, tile, 1)) {
            if (blockIdx.x >= ra.team_blocks) return;
            workers = ra.team_blocks * kWaves;
            team = kTeam;
            me = threadIdx.x % (kTeam * kWave);
            at /= kTeam;
        }
        // the vectors (in 64s) of these 64 records' pages
        const uint64_t v = (uint64_t)g.pages * ((tile + kWave - 1) / kWave);
        const uint32_t most = 1u << 25, all = lane32(wave_scan32(v < most ? (uint32_t)v : most), kWave - 1);
        // a part: 64 U vectors, or more when there are many
        const uint32_t unit = kUnit * team;
        const float even = (float)all * (team == 1 ? ra.even : ra.team_even);
        uint32_t part_vecs = (even < (float)(0x40000000 / unit) ? (uint32_t)even + 1 : 0x40000000 / unit) * unit;
        uint32_t parts = (tile + part_vecs - 1) / part_vecs;
        if (team > 1 && parts > 1) part_vecs = ((tile + parts - 1) / parts + unit - 1) / unit * unit;   // of equal size
        const uint64_t count = (uint64_t)g.pages * parts;
        int64_t end = __ballot(count >> 25) == 0 ? (int64_t)wave_scan32((uint32_t)count) : (int64_t)wave_scan(count);
        int64_t ends = 0;                                  // lane i: parts of wavefront i's records
        if (SHARE) {
            shared->rec[threadIdx.x] = g;
            shared->end[threadIdx.x] = end;
            shared->parts[threadIdx.x] = parts;
            shared->part_vecs[threadIdx.x] = part_vecs;
            __syncthreads();
            if (lane < (uint32_t)kWaves) ends = shared->end[lane * kWave + kWave - 1];
        }
        for (int c = 0; c < (SHARE ? kWaves : 1); ++c) {
            const int64_t total = (SHARE ? lane64(ends, c) : lane64(end, kWave - 1)) * L;
            if (SHARE) {
                if (at >= total) {
                    at -= total;
                    continue;
                }
                g = shared->rec[c * kWave + lane];
                end = shared->end[c * kWave + lane];
                parts = shared->parts[c * kWave + lane];
                part_vecs = shared->part_vecs[c * kWave + lane];
            }
            for (; at < total; at += workers / team) {
                const GridArgs &a = fresh_args();
                const uint64_t rem = at < INT32_MAX ? fd_div(a.fd_L, (uint32_t)at) : (uint64_t)at / L;
                const uint32_t l = (uint32_t)(at - (int64_t)rem * L);
                const int r = __builtin_ctzll(__ballot(end > rem));
                const uint32_t r_parts = lane32(parts, r);
                const uint64_t in = rem - (lane64(end, r) - lane64(g.pages, r) * r_parts);
                uint32_t j = (uint32_t)in, part = 0;
                if (r_parts > 1) {
                    j = in <= ~0u ? (uint32_t)in / r_parts : (uint32_t)(in / r_parts);
                    part = (uint32_t)(in - (uint64_t)j * r_parts);
                }
                uint32_t sa = lane32(g.sa, r), left = lane32(g.n, r);
                const int64_t t_idx = lane64(g.t_idx, r) + j;
                GridPart w;
                w.pos = lane32(g.pos, r);
                if (j > 0) {
                    const uint32_t skip = j * T - sa;
                    sa = 0;
                    left -= skip;
                    w.pos += skip;
                }
                const uint32_t ntok = left < T - sa ? left : T - sa;
                w.o_off = lane64(g.o_off, r);
                w.sa = sa;
                w.ntok = ntok;
                w.R = unit_slots<MODE>(sa, ntok, a.slot_shift) * a.fd_hv.d;
                const uint32_t vecs = w.R * a.C;
                const uint32_t size = lane32(part_vecs, r);
                w.kb = part * size;
                if (w.kb >= vecs) continue;
                w.ke = vecs - w.kb < size ? vecs : w.kb + size;
                // the page ids of both sides: the other side's pages of this page's
                // tokens, the first 64 of them, one per lane
                const uint32_t tpage = (uint32_t)cload(a.t_pt + t_idx);
                uint32_t jo0 = 0, K = 1, opid = 0, bits = 0;
                if (kPool) {
                    jo0 = fd_div(a.fd_To, w.pos);
                    K = fd_div(a.fd_To, w.pos + ntok - 1) - jo0 + 1;
                    if (lane < K) {
                        const int64_t idx = w.o_off + jo0 + lane;
                        if (idx < 0 || idx >= a.o_len) bits = KVX_DERR_PT_RANGE;
                        else opid = (uint32_t)a.o_pt[idx];
                    }
                }
                if (tpage >= a.t_N) {
                    if (lane == 0 && a.err) atomicOr(a.err, OP == OP_GATHER ? KVX_DERR_SRC_PAGE : KVX_DERR_DST_PAGE);
                    continue;
                }
                w.t = a.t_base + (int64_t)l * a.t_l + (int64_t)tpage * a.t_p + (uint64_t)sa * a.t_t * 16;
                const auto from_lane = [&](uint32_t jo, bool valid) {
                    const uint32_t i = valid ? jo - jo0 : 0;
                    uint32_t pg = (uint32_t)__shfl((int)opid, i < kWave ? i : 0, kWave);
                    if (i >= kWave) pg = other_page(a, w.o_off + jo);      // more pages than lanes
                    return pg;
                };
                if (!kPool) {
                    const uint64_t run = (uint64_t)lane32(g.n_block, r) * a.fd_hv.d;   // vectors of one kv component's block
                    w.o = a.o_base + w.o_off + ((uint64_t)l * a.C * run + (uint64_t)w.pos * a.fd_hv.d) * 16;
                    w.o_c = run * 16;
                    copy_part<OP, MODE, true, HOST, U>(a, w, me, team * kWave, from_lane);
                    continue;
                }
                if (lane < K && opid >= a.o_N && !bits) bits = KVX_DERR_SRC_PAGE;
                if (bits) {
                    opid = ~0u;
                    if (a.err) atomicOr(a.err, bits);
                }
                w.o = a.o_base + (int64_t)l * a.o_l;
                w.o_c = (uint64_t)a.o_c * 16;
                if (K == 1) {
                    const uint32_t pg = lane32(opid, 0);
                    if (pg == ~0u) continue;
                    w.o += (int64_t)pg * a.o_p + (uint64_t)(w.pos - jo0 * a.fd_To.d) * a.o_t * 16;
                    copy_part<OP, MODE, true, HOST, U>(a, w, me, team * kWave, from_lane);
                } else {
                    copy_part<OP, MODE, false, HOST, U>(a, w, me, team * kWave, from_lane);
                }
            }
            at -= total;
        }
        if (SHARE) __syncthreads();                         // the next records take the place of these
    }
}

template <int OP, SweepMode MODE, bool HOST, int U>
__global__ void __launch_bounds__(kBlock) kvx_parts_kernel(GridArgs) {
    copy_parts<OP, MODE, HOST, U, kBlock, false>(nullptr);
}

// The same for more than 64 records.  (Six wavefronts per SIMD: with 81 registers for
// head-major rows it had five, 4000 records of 1-8 tokens 1139 us : 1039.)
template <SweepMode MODE>
constexpr int kShareBlock = MODE == ROWS_T || MODE == ROWS_H ? kBlock : KVX_SHARE_BLOCK;
template <int OP, SweepMode MODE, bool HOST, int U>
__global__ void __launch_bounds__(kShareBlock<MODE>, MODE == ROWS_H && U == KVX_PARTS_UNROLL
                                                         ? KVX_SHARE_ROWS_BLOCKS_PER_CU : 1)
kvx_shared_parts_kernel(GridArgs) {
    __shared__ Records<kShareBlock<MODE>> shared;
    copy_parts<OP, MODE, HOST, U, kShareBlock<MODE>, true>(&shared);
}

// Wavefronts, of an XCD's W, that take a unit of so many pieces together: as many
// as it has pieces, or fewer in turns where that leaves fewer of the W idle.
__host__ __device__ inline uint32_t team_size(uint32_t pieces, uint32_t W) {
    if (pieces <= W / 8) return pieces;
    uint32_t size = W, used = 0;
    for (uint32_t s = 1; s <= 8; ++s) {
        const uint32_t z = (pieces + s - 1) / s;
        if (z > W) continue;
        const uint32_t u = W / z * z;
        if (u > used + W / 16) used = u, size = z;
    }
    return size;
}

// Persistent grid that keeps the sweep's order, for calls of long records.
// XCD x copies the units x, x + 8, ...; a team of its wavefronts takes a unit
// together, 64 vectors (1 KiB) each, and goes on to the unit `teams` further,
// so that what is in flight slides through a few pages per XCD.  Two things
// keep it so:
// - every lane plans one unit of its wavefront ahead (record by binary search
//   in LDS, page ids, addresses), 64 units at a time, so that a piece costs
//   the wavefront a few lane reads instead of a search (which ran at 4.8
//   TB/s);
// - a workgroup barrier before each piece: without it the wavefronts drift
//   apart and the rate falls back to that of pages per wavefront (8528 us
//   below; 7146 us with it).
// A team member's piece turns from unit to unit, so that units that are not
// full cost everybody the same.  Units of more pieces than an XCD has
// wavefronts are taken in turns.
// Against a page per wavefront (us): 32 prompts of 36 x 8 x 128, 256 KiB
// pages, 43.7 GB, 8591 -> 7146 (6.1 TB/s; 6957 -> 6998 on pools that suit the
// grid); 1500 tokens 92 -> 80.9; 72 KiB pages 4941 -> 4751; a scatter from a
// buffer into 64 KiB pages of 6.2 GB 1190 -> 1060.
template <int OP, SweepMode MODE, int B, int U>
__global__ void __launch_bounds__(B) kvx_order_kernel(GridArgs) {
    constexpr bool HOST = false;                   // (never over the link)
    constexpr bool kPool = OP == OP_TRANSFER;
    __shared__ Records<B> shared;
    int64_t *const s_end = shared.end;             // end of record i's pages among the chunk's
    GridRec *const s_rec = shared.rec;
    __shared__ int64_t s_sum[B / kWave];
    __shared__ uint32_t s_max[B / kWave];
    const uint32_t lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t x = blockIdx.x & 7u, w = wave * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const uint32_t W = (gridDim.x >> 3) * (B / kWave);
    const int32_t n_reqs = fresh_args().n_reqs;
    {
        // Whether the first 64 records are worth the order.
        const GridArgs &a = fresh_args();
        GridRec g;
        (void)grid_record<OP>(a, load_raw(a, lane), g);
        const uint32_t T = a.fd_Tt.d, To = a.fd_To.d;
        // Whether the other side's pages begin between units, or between pieces
        // (of units that are not taken in turns).
        const uint32_t ahead = (uint32_t)g.pos + T - (uint32_t)g.sa;
        const bool units = ahead == fd_div(a.fd_Tt, ahead) * T && To % T == 0;
        const bool between = a.granule > 0 && ((ahead | T | To) & (a.granule - 1)) == 0;
        const uint32_t n = g.pages && (!kPool || units || between) ? (uint32_t)g.n : 0;
        const uint64_t tokens = (uint64_t)lane64(wave_scan(n), kWave - 1);
        const uint64_t pages = (uint64_t)lane64(wave_scan((uint64_t)g.pages), kWave - 1);
        const uint32_t token_vecs = a.fd_hv.d * a.C;
        if (!(4 * tokens >= KVX_ORDER_QUARTERS * pages * T &&
              tokens * token_vecs * a.fd_L.d >= (uint64_t)W * 8 * KVX_ORDER_TURNS * kWave)) {
            if (n_reqs > kWave) copy_parts<OP, MODE, HOST, U, B, true>(&shared);
            else copy_parts<OP, MODE, HOST, U, B, false>(nullptr);
            return;
        }
    }
    for (int32_t r0 = 0; r0 < n_reqs; r0 += B) {
        const GridArgs &ra = fresh_args();
        const uint32_t L = ra.fd_L.d, T = ra.fd_Tt.d;
        GridRec g;
        const uint32_t bad = grid_record<OP>(ra, load_raw(ra, r0 + threadIdx.x), g);
        if (bad && blockIdx.x == 0 && ra.err) atomicOr(ra.err, bad);
        s_rec[threadIdx.x] = g;
        // vectors of the record's largest page
        uint32_t most = (g.pages == 0 ? 0 : (uint32_t)g.n < T ? (uint32_t)g.n : T) * ra.fd_hv.d * ra.C;
        int64_t end = (int64_t)wave_scan((uint64_t)g.pages);
        most = wave_max(most);
        if (lane == kWave - 1) {
            s_sum[wave] = end;
            s_max[wave] = most;
        }
        __syncthreads();
        {
            // the wavefronts before this one
            const uint64_t sums = wave_scan(lane < B / kWave ? (uint64_t)s_sum[lane] : 0);
            most = wave_max(lane < B / kWave ? s_max[lane] : 0);
            if (wave) end += lane64((int64_t)sums, wave - 1);
        }
        s_end[threadIdx.x] = end;
        __syncthreads();
        const int64_t units = lane64(s_end[B - 1], 0) * L;
        most = __builtin_amdgcn_readfirstlane(most);
        // A team of `size` wavefronts of the XCD copies a unit, each of them
        // every size-th piece of it.
        const uint32_t pieces = (most + kWave - 1) / kWave, size = team_size(pieces, W);
        const uint32_t turns = pieces > size ? (pieces + size - 1) / size : 1;
        const uint32_t teams = pieces ? W / size : 1, team = pieces ? w / size : 1;
        const uint32_t p0 = w - team * size, turn = (size / 2 + size / 8) | 1;
        const int64_t n0 = units > x ? (units - x + 8ll * teams - 1) / (8ll * teams) : 0;
        for (int64_t b = 0; b < n0; b += kWave) {
            // Each lane plans one unit.
            const GridArgs &a = fresh_args();
            const int64_t i = b + lane, at = (team + i * teams) * 8 + x;
            bool ok = at < units && team < teams, one = true;
            int64_t t_off = 0, o_off = 0, o_pt = 0;
            uint64_t o_c = 0;
            uint32_t kb = 0, R = 0, sa = 0, ntok = 0, pos = 0, l = 0;
            if (ok) {
                const int64_t n = units < INT32_MAX ? (int64_t)fd_div(a.fd_L, (uint32_t)at) : at / L;
                l = (uint32_t)(at - n * L);
                uint32_t r = 0;                    // first record whose pages end past n
#pragma unroll
                for (uint32_t step = B / 2; step; step >>= 1)
                    if (s_end[r + step - 1] <= n) r += step;
                const GridRec g = s_rec[r];
                const uint32_t j = (uint32_t)(n - (r ? s_end[r - 1] : 0));
                uint32_t left = (uint32_t)g.n;
                sa = g.sa;
                pos = g.pos;
                if (j) {
                    const uint32_t skip = j * T - sa;
                    sa = 0;
                    left -= skip;
                    pos += skip;
                }
                ntok = left < T - sa ? left : T - sa;
                R = ntok * a.fd_hv.d;
                const uint32_t vecs = R * a.C;
                kb = (p0 + (uint32_t)i * turn) % size * kWave;
                ok = kb < vecs;
                if (ok) {
                    const uint32_t tpage = (uint32_t)a.t_pt[g.t_idx + j];
                    o_pt = g.o_off;
                    uint32_t jo0 = 0, opage = 0, bits = 0;
                    if (kPool) {
                        // the other side's pages of the piece's tokens (of the
                        // whole unit when the piece is one of several)
                        const uint32_t ke = (kb + kWave < vecs ? kb + kWave : vecs) - 1;
                        const bool c0 = kb >= R, c1 = ke >= R;
                        uint32_t t0 = 0, t1 = ntok - 1;
                        if (c0 == c1 && turns == 1) {
                            t0 = fd_div(a.fd_hv, c0 ? kb - R : kb);
                            t1 = fd_div(a.fd_hv, c0 ? ke - R : ke);
                        }
                        jo0 = fd_div(a.fd_To, pos + t0);
                        one = jo0 == fd_div(a.fd_To, pos + t1);
                        const int64_t idx = o_pt + jo0;
                        const bool in = idx >= 0 && idx < a.o_len;
                        if (one) {
                            opage = in ? (uint32_t)a.o_pt[idx] : 0;
                            bits = !in ? KVX_DERR_PT_RANGE : opage >= a.o_N ? KVX_DERR_SRC_PAGE : 0;
                        }
                    }
                    if (tpage >= a.t_N) bits = OP == OP_GATHER ? KVX_DERR_SRC_PAGE : KVX_DERR_DST_PAGE;
                    if (bits) {
                        ok = false;
                        if (a.err) atomicOr(a.err, bits);
                    }
                    t_off = (int64_t)l * a.t_l + (int64_t)tpage * a.t_p + (int64_t)sa * a.t_t * 16;
                    if (kPool) {
                        o_off = (int64_t)l * a.o_l;
                        if (one) o_off += (int64_t)opage * a.o_p + ((int64_t)pos - (int64_t)jo0 * a.fd_To.d) * a.o_t * 16;
                    } else {
                        const uint64_t run = (uint64_t)g.n_block * a.fd_hv.d;    // vectors of one kv component's block
                        o_c = run * 16;
                        o_off = g.o_off + ((int64_t)l * a.C * run + (int64_t)pos * a.fd_hv.d) * 16;
                    }
                }
            }
            // Then the wavefront copies its pieces of the units, in order.
            uint64_t todo = __ballot(ok);
            const uint64_t ones = __ballot(one);
            const GridArgs &ca = fresh_args();
            const int rounds = n0 - b < kWave ? (int)(n0 - b) : kWave;
            const auto piece = [&](int u, GridPart &c) {
                c.t = ca.t_base + lane64(t_off, u);
                c.o = ca.o_base + lane64(o_off, u);
                c.o_c = kPool ? (uint64_t)ca.o_c * 16 : (uint64_t)lane64((int64_t)o_c, u);
                c.R = lane32(R, u);
                c.kb = lane32(kb, u);
                c.ke = c.R * ca.C;
            };
            const auto none = [](uint32_t, bool) { return ~0u; };
            if (turns == 1 && (todo & ~ones) == 0) {
                for (int k = 0; k < rounds; ++k) {
                    __builtin_amdgcn_s_barrier();
                    if (todo == 0) continue;
                    const int u = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    GridPart c;
                    piece(u, c);
                    const char *src;
                    char *dst;
                    if (part_vector<OP, MODE, true>(ca, c, c.kb + lane, none, src, dst)) st16<HOST>(dst, ld16(src));
                }
                continue;
            }
            for (int k = 0; k < rounds; ++k) {
                __builtin_amdgcn_s_barrier();
                if (todo == 0) continue;
                const int u = __builtin_ctzll(todo);
                todo &= todo - 1;
                GridPart c;
                piece(u, c);
                c.o_off = lane64(o_pt, u);
                c.pos = lane32(pos, u);
                const uint32_t vecs = c.ke;
                for (uint32_t i = 0; i < turns && c.kb < vecs; ++i, c.kb += size * kWave) {
                    c.ke = vecs - c.kb < kWave ? vecs : c.kb + kWave;
                    if (!kPool || (ones >> u & 1)) {
                        copy_part<OP, MODE, true, HOST, 1>(ca, c, lane, kWave, none);
                    } else {
                        copy_part<OP, MODE, false, HOST, 1>(ca, c, lane, kWave, [&](uint32_t jo, bool valid) {
                            return valid ? other_page(ca, c.o_off + jo) : ~0u;
                        });
                    }
                }
            }
        }
        __syncthreads();                            // the next chunk reuses the shared state
    }
}

}  // namespace

// The sweep's launch: the pieces of layers x plan pages, in as many launches
// as its workgroups need (KVX_SWEEP_MAX_BLOCKS each).
static int launch_sweep(const Params &p, hipStream_t stream) {
    const Side &d = p.dst, &s = p.src;
    const bool adjacent = (p.H == 1 || (d.s_h == p.row_bytes && s.s_h == p.row_bytes)) &&
                          d.s_t >= (int64_t)p.H * p.row_bytes && s.s_t >= (int64_t)p.H * p.row_bytes;
    const SweepMode mode = p.flat ? RUNS : adjacent ? TOKENS : d.tok_contig ? ROWS_T : ROWS_H;
    typedef void (*SweepFn)(SweepArgs, Params);
#define KVX_SWEEPS(mode)                                                                  \
    {{kvx_sweep_kernel<mode, false, false>, kvx_sweep_kernel<mode, false, true>},          \
     {kvx_sweep_kernel<mode, true, false>, kvx_sweep_kernel<mode, true, true>}}
    static const SweepFn fns[4][2][2] = {KVX_SWEEPS(RUNS), KVX_SWEEPS(TOKENS), KVX_SWEEPS(ROWS_T), KVX_SWEEPS(ROWS_H)};
#undef KVX_SWEEPS
    const bool sparse = p.plan_slots < d.T;
    const SweepFn fn = fns[mode][p.dst_host ? 1 : 0][sparse];
    constexpr int64_t SB = KVX_SWEEP_SLOT_BLOCK;
    const int64_t page_slots = mode == ROWS_H ? ((int64_t)d.T + SB - 1) / SB * SB : d.T;
    // bytes from a page's first copied row to the end of its last one
    const auto extent = [&](const Side &x) {
        return (page_slots - 1) * x.s_t + (p.C - 1) * x.s_c + (p.H - 1) * x.s_h + p.row_bytes;
    };
    SweepArgs a{};
    a.slots = p.slots;
    // the workgroups of a page: one per piece of as many slots as a page copies
    const int64_t used = !sparse ? page_slots
                         : mode == ROWS_H ? ((int64_t)p.plan_slots + SB - 1) / SB * SB : p.plan_slots;
    a.ppt = make_fastdiv(sweep_pieces(p, used));
    a.pages = make_fastdiv((uint32_t)p.plan_pages);
    const auto fits = [&](const Side &x) {
        return extent(x) <= INT32_MAX && x.s_l / 16 <= UINT32_MAX && x.s_p / 16 <= UINT32_MAX;
    };
    a.general = !(fits(d) && fits(s));
    a.d_pt = d.pt;
    a.s_pt = s.pt;
    a.d_last = (uint32_t)d.pt_len - 1;
    a.s_last = (uint32_t)s.pt_len - 1;
    a.d_T = d.T;
    a.s_T = s.T;
    a.d_lastp = (uint32_t)d.N - 1;
    a.s_lastp = (uint32_t)s.N - 1;
    a.fd_To = p.fd_To;
    a.fd_hv = make_fastdiv((uint32_t)(p.H * p.vpr));
    a.C = p.C;
    a.d_t = (uint32_t)d.s_t;
    a.s_t = (uint32_t)s.s_t;
    a.d_c = (uint32_t)d.s_c;
    a.s_c = (uint32_t)s.s_c;
    a.d_l = (uint32_t)(d.s_l / 16);
    a.d_p = (uint32_t)(d.s_p / 16);
    a.s_l = (uint32_t)(s.s_l / 16);
    a.s_p = (uint32_t)(s.s_p / 16);
    a.d_base = d.base;
    a.s_base = s.base;
    a.H = p.H;
    a.vpr = p.vpr;
    a.d_h = (uint32_t)d.s_h;
    a.s_h = (uint32_t)s.s_h;
    a.fd_H = p.fd_H;
    a.fd_vpr = p.fd_vpr;
    const int64_t n_check = ((p.plan_pages > p.n_reqs ? p.plan_pages : p.n_reqs) + kWave - 1) / kWave;
    const int64_t total = (int64_t)p.L * p.plan_pages;
    int64_t per = KVX_SWEEP_MAX_BLOCKS / a.ppt.d;                  // page slots per launch
    if (per > 8) per &= ~(int64_t)7;
    for (int64_t s0 = 0; s0 < total; s0 += per) {
        a.slot0 = (uint32_t)s0;
        a.n_slots = (uint32_t)(total - s0 < per ? total - s0 : per);
        a.checks = s0 ? 0 : (uint32_t)((n_check < 1024 ? n_check : 1024) + 7) / 8 * 8;
        hipLaunchKernelGGL(fn, dim3(a.checks + a.n_slots * a.ppt.d), dim3(kWave), 0, stream, a, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Compute units of the current device, asked for once per device.
hipError_t device_cus(int *cus) {
    static std::atomic<int> seen[64];
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 64 && (*cus = seen[dev].load(std::memory_order_relaxed)) > 0) return hipSuccess;
    const hipError_t q = hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (q == hipSuccess && dev < 64) seen[dev].store(*cus, std::memory_order_relaxed);
    return q;
}

// log2 of the slots per block of a head-major tiling side's vector order: blocks
// of KVX_SLOT_BLOCK slots, and of rows narrower than a 128-byte line as many more
// as end with one, up to 8.  A page's narrow rows are written by several
// wavefronts, and a line whose halves come from two of them is written twice.
// 17 records of 900-1100 tokens, 330 MB, blocks of 2 and of 8 (4 for 96 bytes), us:
// 8 heads of 48 bytes 87 and 48, of 80 bytes 126 and 70, 5 of 112 bytes 105 and 70, 5 of
// 96 bytes 75 and 67; a workgroup per page, blocks of 2, took 65, 93, 89 and 71.  With
// rows of whole lines larger blocks only add masked slots to short records (2000 of
// 1-4 tokens, 8 heads of 256 bytes: 305 us with blocks of 2, 361 of 4, 556 of 8).
static uint32_t slot_shift(const Params &p, int32_t T) {
    uint32_t sb = (uint32_t)__builtin_ctz(KVX_SLOT_BLOCK);
    while (p.row_bytes < 128 && sb < 3 && ((p.row_bytes << sb) & 127)) ++sb;
    // (a page's vectors, whole blocks of them, are numbered with 31 bits)
    const int64_t slots = ((((int64_t)T - 1) >> sb) + 1) << sb;
    return slots * p.C * p.H * p.vpr <= INT32_MAX ? sb : (uint32_t)__builtin_ctz(KVX_SLOT_BLOCK);
}

// The launch of an unplanned call.
template <int OP>
static int launch_grid(const Params &p, hipStream_t stream) {
    const Side &t = OP == OP_GATHER ? p.src : p.dst, &o = OP == OP_GATHER ? p.dst : p.src;
    int cus = 0;
    const hipError_t e = device_cus(&cus);
    if (e != hipSuccess) return e;
    const int64_t row = p.row_bytes;
    const auto adjacent = [&](const Side &x, bool pool) {
        return !pool || ((p.H == 1 || x.s_h == row) && x.s_t >= (int64_t)p.H * row);
    };
    const bool t_adjacent = adjacent(t, true);
    const SweepMode mode = p.flat ? RUNS : !t_adjacent ? ROWS_H : adjacent(o, OP == OP_TRANSFER) ? TOKENS : ROWS_T;
    typedef void (*GridFn)(GridArgs);
    constexpr int B = KVX_ORDER_BLOCK, U = KVX_PARTS_UNROLL, UL = KVX_LINK_UNROLL;
#define KVX_MODES(kernel, ...)                                                                                 \
    {kernel<OP, RUNS, __VA_ARGS__>, kernel<OP, TOKENS, __VA_ARGS__>, kernel<OP, ROWS_T, __VA_ARGS__>,          \
     kernel<OP, ROWS_H, __VA_ARGS__>}
    static const GridFn order_fns[2] = {kvx_order_kernel<OP, RUNS, B, U>, kvx_order_kernel<OP, TOKENS, B, U>};
    // [more than 64 records][mode], and over the link [into host memory] of those
    static const GridFn parts_fns[2][4] = {KVX_MODES(kvx_parts_kernel, false, U),
                                           KVX_MODES(kvx_shared_parts_kernel, false, U)};
    static const GridFn link_fns[2][2][4] = {
        {KVX_MODES(kvx_parts_kernel, false, UL), KVX_MODES(kvx_shared_parts_kernel, false, UL)},
        {KVX_MODES(kvx_parts_kernel, true, UL), KVX_MODES(kvx_shared_parts_kernel, true, UL)}};
#undef KVX_MODES
    GridArgs a{};
    a.reqs = p.reqs;
    a.err = p.err;
    a.n_reqs = p.n_reqs;
    a.t_base = t.base;
    a.o_base = o.base;
    a.t_l = t.s_l;
    a.t_p = t.s_p;
    a.o_l = o.s_l;
    a.o_p = o.s_p;
    a.t_pt = t.pt;
    a.o_pt = o.pt;
    a.t_len = t.pt_len;
    a.o_len = o.pt_len;
    a.cap_bytes = o.cap_bytes;
    a.token_bytes = (int64_t)p.L * p.C * p.H * row;
    a.t_N = (uint32_t)t.N;
    a.o_N = (uint32_t)o.N;
    a.C = p.C;
    a.elem_shift = (uint32_t)__builtin_ctz((unsigned)p.elem_bytes);
    a.t_c = (uint32_t)(t.s_c / 16);
    a.t_t = (uint32_t)(t.s_t / 16);
    if (OP == OP_TRANSFER) {
        a.o_c = (uint32_t)(o.s_c / 16);
        a.o_t = (uint32_t)(o.s_t / 16);
    } else {
        a.o_t = p.H * p.vpr;
    }
    a.t_h = (uint32_t)(t.s_h / 16);
    a.o_h = OP == OP_TRANSFER ? (uint32_t)(o.s_h / 16) : (uint32_t)p.vpr;
    a.slot_shift = slot_shift(p, t.T);
    a.fd_vpr = p.fd_vpr;
    a.fd_H = p.fd_H;
    a.fd_Tt = p.fd_Tt;
    a.fd_To = p.fd_To;
    a.fd_hv = make_fastdiv((uint32_t)(p.H * p.vpr));
    a.fd_L = make_fastdiv((uint32_t)p.L);
    const uint32_t pieces = (uint32_t)(((int64_t)t.T * p.C * p.H * p.vpr + kWave - 1) / kWave);
    a.granule = team_size(pieces, (cus + 7) / 8 * (B / kWave)) < pieces ? 0 : kWave;
    while (a.granule > 1 && a.granule / 2 * (a.fd_hv.d % kWave) % kWave == 0) a.granule /= 2;
    const bool link = p.src_host || p.dst_host;
    const int64_t page_vecs = (int64_t)t.T * p.C * p.H * p.vpr;
    const bool rows = mode == ROWS_T || mode == ROWS_H;
    a.team_min = rows && !link ? (uint64_t)cus * KVX_PARTS_BLOCKS_PER_CU * 4 * KVX_TEAM_KIB * kWave : ~0ull;
    const bool order = !rows && !link && t.pt_len >= (int64_t)KVX_ORDER_PAGES * p.n_reqs &&
                       page_vecs >= (int64_t)KVX_ORDER_PIECES * kWave;
    const bool share = p.n_reqs > kWave;
    const int threads = order ? B : share && !rows ? KVX_SHARE_BLOCK : kBlock;
    int blocks = (cus + 7) / 8 * 8;
    if (!order)
        blocks = cus * (link ? KVX_LINK_BLOCKS_PER_CU * kBlock / threads
                        : !share ? KVX_PARTS_BLOCKS_PER_CU : rows ? KVX_SHARE_ROWS_BLOCKS_PER_CU : KVX_SHARE_BLOCKS_PER_CU);
    // the vectors of all records, were they like these 64, over the parts aimed at
    const float per_64 = 64.f * p.L * ((p.n_reqs + kWave - 1) / kWave), waves = (float)blocks * (threads / kWave);
    a.even = link ? per_64 / (float)(KVX_LINK_PARTS * kWave * UL) : per_64 / (waves * KVX_GRID_PARTS * kWave * U);
    a.team_blocks = (uint32_t)std::min(blocks, cus * KVX_TEAM_BLOCKS_PER_CU);
    a.team_even = per_64 / ((float)a.team_blocks * 4 * KVX_TEAM_PARTS * kWave * 4 * U);
    const GridFn fn = order ? order_fns[mode] : link ? link_fns[p.dst_host ? 1 : 0][share][mode] : parts_fns[share][mode];
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(threads), 0, stream, a);
    return hipGetLastError();
}

// Sweep when the host chose it (p.sweep), else a persistent grid: as
// many workgroups as the device holds at once.
int launch(const Params &p, hipStream_t stream) {
    if (p.sweep) return launch_sweep(p, stream);
    switch (p.op) {
    case OP_TRANSFER: return launch_grid<OP_TRANSFER>(p, stream);
    case OP_GATHER: return launch_grid<OP_GATHER>(p, stream);
    default: return launch_grid<OP_SCATTER>(p, stream);
    }
}

}  // namespace kvx
