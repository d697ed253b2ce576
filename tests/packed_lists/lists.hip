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
// (choose_list), and whether candidates are found by division; returns the window steps.
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
    *division = packed_by_division(a, *total_out, align);
    return steps;
}

extern "C" void packed_place(int C, int S, int Hq, int Hkv, int r0, int *b, int *first)
{
    const Walk w = walk_by_division(problem(C, S, Hq, Hkv), r0);
    *b = w.b, *first = w.first;
}
