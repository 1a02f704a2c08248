"""The lists of arrays that the library copies or permutes in one launch hold a
fixed number: one more is left out, noted, and refused by the launch, and
nothing is written past the end (host)."""
import ctypes

from host_arith import compile_host

SOURCE = """
#include <hip/hip_runtime.h>
#include "gcb_internal.h"
struct Guarded { gcb::CopyList c; long mark = 77; gcb::PermuteList p; long mark2 = 78; };
extern "C" int lists(int copies, int permutes) {
    Guarded g;
    double a = 0.0, b = 0.0;
    for (int i = 0; i < copies; ++i) g.c.add(&a, &b, 8);
    for (int i = 0; i < permutes; ++i) g.p.add(&a, &b);
    if (g.mark != 77 || g.mark2 != 78) return -1;
    return (g.c.n == (copies < gcb::CopyList::kMax ? copies : gcb::CopyList::kMax)) +
           2 * (g.p.n == (permutes < gcb::PermuteList::kMax ? permutes : gcb::PermuteList::kMax)) +
           4 * g.c.over + 8 * g.p.over;
}
"""


def test_lists_end(tmp_path):
    lib = compile_host(str(tmp_path), SOURCE)
    lib.lists.restype = ctypes.c_int
    assert lib.lists(0, 0) == 3
    assert lib.lists(12, 10) == 3       # the 3D state with q/m and ids; the permuted state
    assert lib.lists(13, 10) == 3 + 4
    assert lib.lists(12, 11) == 3 + 8
    assert lib.lists(20, 20) == 3 + 4 + 8
