// Interface of the one-launch opening of a linear layer's operands (open_recode.hip) to the entry points (linear.hip).
#pragma once
#include "common.h"

// A sharing x masked by a, both of [rows][K] words at src[r * row_stride + k * k_stride] (+ tap * tap_stride for a filter's
// taps), and the digit planes formed of them, with e_i = x_i - a_i exchanged on the way (e = e_0 + e_1):
//   folded calls: dst[0] of x_0 + e_1, dst[1] of e;
//   plain calls:  dst[0] of e, mask_dst[i] of a_i (with add_open: mask_dst[0] of a_0 + e).
struct OpenSet {
    const u64 *x[2], *a[2];
    u8 *dst[2], *mask_dst[2];
    int add_open;
    long long row_stride, k_stride, src_batch_stride, tap_stride;      // words; one of the first two is 1
    long long digit_stride, dst_batch_stride;              // bytes
    int rows, plane_rows, K, KB_tap, ntaps, KB_total, batch;      // plane rows and k blocks past the operand's own: zero
    unsigned gx, gy, first;                                // filled by the launcher: tiles along rows and k, number of the first one
    int kbt;                                               // filled by the launcher: k blocks of a tile where k is contiguous, else 0
};
constexpr int kMaxOpenSets = 2;
// bytes of receive buffers the launch needs at least, and those it can use
constexpr size_t kOpenBoxBytes = 16384;
// several taps only with contiguous rows
inline bool can_open(const OpenSet& s) { return s.row_stride == 1 || (s.k_stride == 1 && s.ntaps == 1); }
int launch_open_recode(mpc_ctx* c, hipStream_t st, const OpenSet* sets, int count, bool plain, u8* box, size_t box_bytes);
