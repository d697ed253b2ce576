// The arithmetic of the packed lists (pskv_packed.hpp) for a host test: the kernels' own functions, compiled for the host.
#include "pskv_packed.hpp"

using namespace pskv;

static Args problem(int C, int S, int Hq, int Hkv)
{
    Args a = {};
    a.B = a.C = C, a.Np = 1, a.S = S, a.Hq = Hq, a.Hkv = Hkv, a.G = Hq / Hkv;
    a.div_g = make_fastdiv((unsigned)a.G), a.div_s = make_fastdiv((unsigned)S);
    return a;
}

// The list's rows and alignment, as a kernel with room for `most` window steps and `waves` wavefronts to a list chooses it
// (choose_list), and whether every run is a full candidate's; returns the window steps.
extern "C" int packed_list(int C, int S, int Hq, int Hkv, const int *len, int most, int tiles, int waves, int *total_out, int *align_out, int *division)
{
    const Args a = problem(C, S, Hq, Hkv);
    int total = 0, total32 = 0;
    for (int b = 0; b < C; ++b) {
        total += packed_run(a, len[b], 1);
        total32 += packed_run(a, len[b], kBlockRows);
    }
    bool dense;
    const int steps = packed_steps(a, most, dense);
    const int align = steps == 1   ? packed_align<1>(a, dense, tiles, waves, total, total32)
                      : steps == 2 ? packed_align<2>(a, dense, tiles, waves, total, total32)
                                   : packed_align<3>(a, dense, tiles, waves, total, total32);
    *total_out = align == 1 ? total : total32;
    *align_out = align;
    *division = packed_even(a, *total_out, align);
    return steps;
}

// The candidate of row r0 of a list whose runs are all full candidates', and that one's first row.
extern "C" void packed_place(int C, int S, int Hq, int Hkv, int align, int r0, int *b, int *first)
{
    const Args a = problem(C, S, Hq, Hkv);
    const Walk w = walk_even(a, make_fastdiv((unsigned)packed_run(a, S, kBlockRows)), align, r0);
    *b = w.b, *first = w.first;
}

// One block: its first candidate, that one's first row, last row, window width and `wide`; the window's first 96 entries; and what the
// walk is left at (in: what it begins at).
extern "C" void packed_walk(int C, int S, int Hq, int Hkv, const int *len, int r0, int total, int align, int span, int (&walk)[3], int (&out)[5], unsigned (&window)[96])
{
    const Args a = problem(C, S, Hq, Hkv);
    Walk w = {walk[0], walk[1], walk[2]};
    for (int l = 0; l < 96; ++l)
        window[l] = l;
    const BlockSpan x = walk_block(a, w, r0, total, align, span, C, [&](int b) { return b < C ? len[b] : (__builtin_trap(), 0); }, [&](int n, int at) {
        for (int l = 0; l < 96; ++l)
            window[l] = enter_window(window[l], l, n, at);
    });
    for (int l = x.width; x.width > 0 && l < 96; ++l)
        window[l] = window[(x.width - 1) % 96];
    walk[0] = w.b, walk[1] = w.first, walk[2] = w.len;
    out[0] = x.b, out[1] = x.first, out[2] = x.last, out[3] = x.width, out[4] = x.wide;
}
