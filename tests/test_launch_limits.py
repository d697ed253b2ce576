"""A HIP launch holds fewer than 2^32 work-items per dimension.  What the vector kernels can be launched for
is served: where a matrix-core kernel's grid, of larger workgroups, would not fit, they take the problem.
Checked on the host (see launch_notes)."""
from paper_2603_13420_amd import binding as pk
import launch_notes as notes

MOST = 1 << 24                    # workgroups of 256 from which on a launch does not fit


def case(call, dtype, D, groups, Np=1, S=1, P=8):
    """groups (candidate, KV head) pairs of one position each."""
    return notes.case(call, dtype, D, groups // 16, P, S, 16, 16, Np or groups // 16)


def test_large_grids_go_to_kernels_that_can_be_launched(tmp_path):
    # bwd: one unit of 256 threads per pair, for fp32 together with the dq blocks of 16 rows each
    # fwd, Np instructions of one candidate each: one 16-row block per pair
    cases = [(case("bwd", "bf16", 64, MOST - 16), 256), (case("bwd", "bf16", 64, MOST), 64),
             (case("bwd", "f32", 64, MOST - MOST // 16), 256), (case("bwd", "f32", 64, MOST), 64), (case("bwd", "f32", 128, MOST), 64),
             (case("fwd", "f32", 64, MOST - 16, Np=0), 256), (case("fwd", "f32", 128, MOST, Np=0), 64),
             (case("fwd", "bf16", 64, MOST, Np=0), 512)]
    for (c, threads), (rc, launches) in zip(cases, notes.launches(tmp_path, [c for c, _ in cases])):
        assert rc == pk.PSKV_OK and launches, (c, rc, launches)
        assert all(g * b < 1 << 32 for g, b, _ in launches), (c, launches)
        assert launches[-1][1] == threads, (c, launches)
