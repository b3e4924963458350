// Interface of the one-launch opening of a linear layer's operands (open_recode.hip) to the entry points (linear.hip).
#pragma once
#include "common.h"

// A sharing x of two or three parties masked by a, both of [rows][K] words at src[r * row_stride + k * k_stride] (+ tap *
// tap_stride for a filter's taps), and the digit planes formed of them, with e_i = x_i - a_i exchanged on the way (e = sum e_i):
//   kFolded (two parties): dst[0] of x_0 + e_1, dst[1] of e;
//   kMasks:                dst[0] of e, mask_dst[i] of a_i (with add_open: mask_dst[0] of a_0 + e);
//   kOpened:               dst[0] of e alone.
enum class OpenPlanes { kFolded, kMasks, kOpened };
struct OpenSet {
    const u64 *x[3], *a[3];
    u8 *dst[3], *mask_dst[3];
    int add_open;
    long long row_stride, k_stride, src_batch_stride, tap_stride;      // words; one of the first two is 1
    long long digit_stride, dst_batch_stride;              // bytes
    int rows, plane_rows, K, KB_tap, ntaps, KB_total, batch;      // plane rows and k blocks past the operand's own: zero
    unsigned gx, gy, first;                                // filled by the launcher: tiles along rows and k, number of the first one
    int kbt;                                               // filled by the launcher: k blocks of a tile where k is contiguous, else 0
};
constexpr int kMaxOpenSets = 2;
// bytes of receive buffers a workgroup has; the launch needs those of one, and uses as many as it is given
constexpr size_t open_box_bytes(int parties) { return parties == 2 ? 16384 : 24576; }
// tiles of an operand of so many plane rows and k blocks at most, whichever way it is stored, and workgroups of a launch at most
size_t open_most_tiles(int plane_rows, int KB_total, int batch);
size_t open_most_blocks(int parties);
// several taps only with contiguous rows
inline bool can_open(const OpenSet& s) { return s.row_stride == 1 || (s.k_stride == 1 && s.ntaps == 1); }
// whether the launch pays for these operands (their tiles may hold few words)
bool open_pays(int parties, OpenPlanes planes, const OpenSet* sets, int count);
int launch_open_recode(mpc_ctx* c, hipStream_t st, int parties, OpenPlanes planes, const OpenSet* sets, int count, u8* box, size_t box_bytes);
