// Outputs of a one-launch call against its inputs.  Such a launch stores results while other workgroups still read
// operands; the launch-per-step sequences have read an operand everywhere before they write the output.  A call whose
// output shares memory with an input therefore runs step by step, unless (element-wise calls) it is the input's own
// array, element for element: then a word is read by the workgroup that writes it, before it does.
#pragma once
#include <cstddef>
#include <cstdint>

struct Span { const void* p; size_t bytes; int unit; };       // p may be null: no such array

template <int N>
struct Spans {
    Span s[N]; int n = 0;
    void words(const void* p, size_t count) { if (p) s[n++] = Span{ p, 8 * count, 8 }; }
    void bytes(const void* p, size_t count) { if (p) s[n++] = Span{ p, count, 1 }; }
};

template <int NO, int NI>
inline bool outputs_apart(const Spans<NO>& out, const Spans<NI>& in, bool same_index_allowed)
{
    for (int o = 0; o < out.n; ++o)
        for (int i = 0; i < in.n; ++i) {
            const Span &a = out.s[o], &b = in.s[i];
            if (same_index_allowed && a.p == b.p && a.unit == b.unit) continue;
            const uintptr_t pa = (uintptr_t)a.p, pb = (uintptr_t)b.p;
            if (pa < pb + b.bytes && pb < pa + a.bytes) return false;
        }
    return true;
}
