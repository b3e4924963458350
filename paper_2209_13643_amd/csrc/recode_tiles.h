// Which k blocks a workgroup of the tile recoder takes: the second grid index counts (tap, group of four k blocks), taps
// 0 .. ntaps - 1 and, for several taps, the padding behind the last one.  A plain matrix (one tap) takes its padding with
// its last group.  Sets of one launch share the grid of the largest, so indices past a set's own count name no blocks.
#pragma once
#ifdef __HIPCC__
#define MPC_HD __host__ __device__
#else
#define MPC_HD
#endif

struct RecodeTile { int tap, kb0, kb_lim; bool zero; };      // k blocks kb0 .. min(kb0 + 4, kb_lim) - 1 of the tap; zero: the padding

MPC_HD inline int recode_groups(int ntaps, int KB_tap, int KB_total) { return ((ntaps == 1 ? KB_total : KB_tap) + 3) / 4; }

MPC_HD inline unsigned recode_tile_count(int ntaps, int KB_tap, int KB_total)
{
    return (unsigned)recode_groups(ntaps, KB_tap, KB_total) * (unsigned)(ntaps + (ntaps > 1 && KB_total > ntaps * KB_tap ? 1 : 0));
}

MPC_HD inline RecodeTile recode_tile(int ntaps, int KB_tap, int KB_total, unsigned by)
{
    RecodeTile t;
    if (ntaps == 1) {                  // without the division, which every workgroup would wait for
        t.tap = 0; t.kb0 = (int)by * 4; t.kb_lim = KB_total; t.zero = false;
        return t;
    }
    const int groups = recode_groups(ntaps, KB_tap, KB_total);
    t.tap = (int)by / groups;
    t.kb0 = ((int)by - t.tap * groups) * 4;
    t.zero = t.tap >= ntaps;
    t.kb_lim = !t.zero ? KB_tap : t.tap == ntaps ? KB_total - ntaps * KB_tap : 0;
    return t;
}
