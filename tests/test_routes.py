"""Which kernel takes a problem, on either side of the lines that the launchers draw, at problems timed through
both (the times stand beside the rules)."""
import pytest

from paper_2603_13420_amd import binding as pk
import launch_notes as notes


def check(tmp_path, call, problems):
    cases = [notes.case(call, "bf16", 128, *p[:-1]) for p in problems]
    for (*_, kernel), c, (rc, got) in zip(problems, cases, notes.launches(tmp_path, cases)):
        assert rc == pk.PSKV_OK and kernel in got[0][2], (c, kernel, got)


def test_dq_kernels(tmp_path):
    # B, P, S, Hq, Hkv, Np, kernel: what is fetched once per pass against what is fetched once per launch
    check(tmp_path, "bwd", [
        (1024, 256, 32, 32, 8, 1, "bwd_dq_resident"), (512, 256, 32, 32, 8, 1, "bwd_dq_resident"),
        (64, 256, 32, 32, 8, 1, "bwd_dq_unit"), (512, 128, 32, 32, 8, 1, "bwd_dq_unit"), (512, 64, 32, 32, 8, 1, "bwd_dq_unit"),
        (512, 256, 30, 28, 4, 1, "bwd_dq_resident"), (128, 256, 144, 32, 8, 1, "bwd_dq_resident"),
        (128, 64, 144, 32, 8, 1, "bwd_dq_unit"), (512, 257, 32, 32, 8, 1, "bwd_dq_unit"),
        (512, 256, 32, 32, 8, 8, "bwd_dq_resident"), (256, 128, 20, 32, 8, 1, "bwd_dq_resident"),
        (512, 128, 8, 32, 32, 1, "bwd_dq_mfma"), (512, 600, 20, 32, 8, 1, "bwd_dq_mfma"),
    ])


def test_forward_own_blocks(tmp_path):
    # rows that fill no whole number of blocks: what their own blocks cost against what the pipelined kernels gain
    check(tmp_path, "fwd", [
        (191, 75, 12, 28, 4, 1, "resident_general"), (94, 81, 21, 32, 8, 1, "resident_general"), (89, 171, 21, 32, 8, 1, "resident_general"),
        (24, 99, 22, 32, 4, 1, "resident_general"), (148, 141, 29, 28, 4, 1, "resident_general"),
        (10, 151, 27, 32, 32, 1, "resident_pipelined"), (274, 153, 27, 32, 8, 1, "resident_pipelined"), (213, 142, 29, 28, 4, 1, "resident_pipelined"),
        (512, 128, 28, 32, 32, 1, "resident_pipelined"), (512, 128, 20, 32, 32, 1, "resident_general"),
        (24, 99, 24, 32, 4, 1, "resident_pipelined"),       # (whole blocks: always)
    ])


def test_forward_candidate_passes(tmp_path):
    check(tmp_path, "fwd", [
        (16, 128, 90, 32, 8, 1, "stream_candidate"), (21, 205, 118, 32, 4, 1, "stream_candidate"), (37, 222, 158, 28, 4, 1, "stream_candidate"),
        (17, 147, 136, 28, 4, 1, "resident_general"), (49, 169, 74, 32, 4, 1, "resident_general"), (247, 145, 45, 32, 8, 1, "resident_general"),
        (161, 164, 113, 32, 4, 1, "resident_general"), (64, 128, 141, 32, 32, 1, "resident_general"),
        (73, 93, 147, 32, 8, 1, "stream_candidate"), (23, 85, 157, 32, 8, 1, "stream_candidate"), (188, 72, 155, 28, 4, 1, "stream_candidate"),
        (161, 164, 112, 32, 4, 1, "stream_candidate"),      # (whole blocks)
        (64, 464, 109, 32, 8, 1, "stream_candidate"), (50, 424, 148, 32, 8, 1, "stream_candidate"), (12, 2018, 156, 32, 32, 1, "stream_pipelined"),
        (34, 1114, 111, 28, 4, 1, "stream_pipelined"), (245, 676, 34, 32, 8, 1, "stream_pipelined"), (43, 603, 113, 40, 40, 1, "stream_general"),
        (300, 700, 13, 32, 8, 1, "stream_general"), (512, 512, 29, 32, 32, 1, "stream_pipelined"),
    ])
