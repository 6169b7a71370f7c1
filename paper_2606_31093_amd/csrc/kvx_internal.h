// kvx_internal.h -- launch parameters shared by the C-ABI layer and the HIP
// kernels of libkvx.  Not part of the public interface (include/kvx.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kvx.h"

#ifndef KVX_SLOT_BLOCK
// Head-major tiling side: slots per block of the vector order in the grid.  The
// tiling side's accesses are runs of this many rows, and the other side's,
// whose consecutive heads are adjacent, fill whole slots.  Blocks of 16: records
// of 1-8 tokens 112 us against 81 (a record's blocks are enumerated whole),
// long records equal.
#define KVX_SLOT_BLOCK 2
#endif
// The same for the sweep into a head-major destination (measured: 16 moves
// the relayout 1.4% faster than 2, 8 and 64 in between; the persistent grid
// loses 3% with blocks of 8).
#ifndef KVX_SWEEP_SLOT_BLOCK
#define KVX_SWEEP_SLOT_BLOCK 16
#endif
// A planned transfer can sweep when its records copy at least this many bytes
// per destination page and layer on average, or at least
// KVX_SWEEP_MIN_DENSE_BYTES and two thirds of a page.  Measured against the
// unplanned launch on the same pools, 28 layers in groups of 4, us: full pages of
// 16 KiB (2 x 128, 2.7 GB) 515 to 606 token-major, 533 to 590 from head-major, 562
// to 602 into it, 576 to 605 both; of 32 KiB 1032 to 1168, 1056 to 1137, 1089 to
// 1139, 943 to 1000; of 64 KiB 923 to 973, 935 to 1160, 861 to 1006, 925 to 1053.
// Pages less than two thirds full get workgroups for what they hold on average
// (kvx_sweep_kernel): 256 KiB pages of 16 and 32 tokens of 64 270 to 318 and 440 to
// 554 us.
#ifndef KVX_SWEEP_MIN_BYTES
#define KVX_SWEEP_MIN_BYTES (64 << 10)
#endif
#ifndef KVX_SWEEP_MIN_DENSE_BYTES
#define KVX_SWEEP_MIN_DENSE_BYTES (12 << 10)
#endif
// Most copying workgroups of one sweep launch; up to 1024 that check the plan come
// on top in the first.  The work-items of a launch (64 per workgroup) must stay
// below 2^32, and are at most 2^31 + 2^16.  A larger transfer takes several launches.
#ifndef KVX_SWEEP_MAX_BLOCKS
#define KVX_SWEEP_MAX_BLOCKS (INT32_MAX / 64)
#endif

namespace kvx {

// Unsigned division by a divisor fixed for a launch, for dividends below
// 2^31: q = floor(n * m / 2^(31 + l)) with l = ceil(log2 d) and
// m = ceil(2^(31 + l) / d).  Exact because m * d - 2^(31 + l) < d <= 2^l,
// so the error term n * (m * d - 2^(31 + l)) / 2^(31 + l) stays below
// n / 2^31 < 1 / d of one quotient step (Granlund and Montgomery,
// "Division by invariant integers using multiplication", PLDI 1994).
struct FastDiv {
    uint32_t d;   // divisor, 1 <= d < 2^31
    uint32_t m;   // ceil(2^(31 + l) / d), l = ceil(log2 d); below 2^32
    uint32_t l;
};

inline FastDiv make_fastdiv(uint32_t d) {
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    return FastDiv{d, (uint32_t)(((1ull << (31 + l)) + d - 1) / d), l};
}

// n / d for n < 2^31 without a branch: n * m / 2^(31 + l) = n / d + n * (m *
// d - 2^(31 + l)) / (d * 2^(31 + l)), and the second term, below n / 2^(31 +
// l) < 2^-l <= 1 / d, cannot reach the next multiple of 1 / d.  Taken as
// 2n * m / 2^(32 + l): one 32-bit high product and a 32-bit shift.
__host__ __device__ inline uint32_t fd_div(const FastDiv &f, uint32_t n) {
    return (uint32_t)(((uint64_t)(n << 1) * f.m) >> 32) >> f.l;
}

// One side of a copy.  A pool side addresses row (l, page, c, slot, h) at
// base + l*s_l + page*s_p + c*s_c + slot*s_t + h*s_h (bytes), with base
// already moved to the first layer, kv component and head the call copies;
// a buffer side addresses row (l, c, i, h) of a request's block at
// base + blk + ((l*C + c)*n + i)*H*row + h*row, with blk the block's byte
// offset.
struct Side {
    char *base;
    int64_t s_l, s_p, s_c, s_t, s_h;
    const int32_t *pt;
    int64_t pt_len;
    int32_t T;        // tokens per page (pool side)
    int32_t N;        // pages (pool side)
    int32_t tok_contig;  // rows of consecutive slots, all copied heads, are adjacent
    int64_t cap_bytes;   // buffer side: bytes addressable from base
};

enum Op : int32_t { OP_TRANSFER = 0, OP_GATHER = 1, OP_SCATTER = 2 };

struct Params {
    Side src, dst;
    const kvx_req *reqs;
    uint32_t *err;
    int32_t n_reqs;
    int32_t op;
    int32_t L, C, H;     // layers, kv components and heads copied
    int32_t row_bytes;   // head_dim * elem_bytes, a multiple of 16
    int32_t vpr;         // 16-byte vectors per row
    int32_t elem_bytes;
    int32_t flat;        // both sides tok_contig: a page is C contiguous runs on both
    int32_t src_host, dst_host;   // the side is pinned host memory
    FastDiv fd_vpr, fd_H, fd_To;
    FastDiv fd_Tt;       // tiling side's page_tokens
    // Sweep launch (a planned pool -> pool transfer): prefix[r] =
    // destination pages of records 0..r-1, slots[q] = page q of the plan.
    // sweep == 0: persistent grid.
    int32_t sweep;
    int64_t plan_pages;
    int32_t plan_slots;  // slots copied per destination page: all, or their average when pages are sparse
    const int64_t *prefix;
    const kvx_plan_slot *slots;
};

// Pieces (workgroups) of a page of page_slots slots in a sweep.
inline uint32_t sweep_pieces(const Params &p, int64_t page_slots) {
    const int64_t vecs = (int64_t)p.C * page_slots * p.H * p.vpr;
    return (uint32_t)((vecs + 63) / 64);
}

// Compute units of the current device.
hipError_t device_cus(int *cus);

// Launch on `stream`; returns a hipError_t value.
int launch(const Params &p, hipStream_t stream);

}  // namespace kvx
