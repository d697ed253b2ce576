"""Which kernel takes a problem, on either side of the lines that the launchers draw, at problems timed through
both (the times stand beside the rules)."""
import pytest

from paper_2603_13420_amd import binding as pk
import launch_notes as notes


def check(tmp_path, call, problems, lens=False):
    """The kernel's whole name, and with "<true>", "<2,1>" or the like its first template arguments.  lens: the call brings lengths."""
    cases = [notes.case(call, "bf16", 128, *p[:-1], lens=lens) for p in problems]
    for (*_, kernel), c, (rc, got) in zip(problems, cases, notes.launches(tmp_path, cases)):
        assert rc == pk.PSKV_OK and notes.named(got[0][2], kernel), (c, kernel, got)


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
    four, eight = "stream_candidate4", "stream_candidate"
    check(tmp_path, "fwd", [
        # rows that fill no whole number of blocks, resident prefixes: the resident general kernel, passes of four and of eight
        (10, 213, 69, 32, 8, 1, four + "<false>"), (35, 70, 66, 32, 4, 1, four + "<false>"), (49, 169, 74, 32, 4, 1, four + "<false>"),
        (199, 162, 53, 28, 4, 1, four + "<false>"), (237, 227, 65, 32, 4, 1, "resident_general"),
        (161, 164, 113, 32, 4, 1, "resident_general"), (203, 206, 41, 28, 4, 1, "resident_general"), (198, 171, 58, 28, 4, 1, "resident_general"),
        (247, 145, 45, 32, 8, 1, "resident_general"), (64, 128, 141, 32, 32, 1, "resident_general"),
        (13, 77, 135, 32, 8, 1, four + "<false>"), (265, 168, 157, 32, 32, 1, "resident_general"), (48, 157, 151, 32, 32, 1, "resident_general"),
        (12, 99, 87, 32, 8, 1, eight + "<false>"), (20, 151, 132, 32, 8, 1, eight + "<false>"), (37, 222, 158, 28, 4, 1, eight + "<false>"),
        (16, 128, 90, 32, 8, 1, eight + "<false>"), (220, 78, 115, 32, 8, 1, four + "<false>"), (14, 94, 77, 32, 8, 1, four + "<false>"),
        # prefixes of their own lengths
        (112, 86, 77, 32, 8, 2, "resident_general"), (48, 69, 123, 32, 8, 2, "resident_general"), (222, 115, 52, 28, 4, 2, "resident_general"),
        (20, 116, 148, 32, 8, 2, eight + "<false>"), (264, 93, 87, 40, 40, 8, four + "<false>"), (186, 157, 87, 32, 8, 2, four + "<false>"),
        # whole blocks, resident prefixes
        (161, 164, 112, 32, 4, 1, four + "<true>"), (300, 128, 120, 32, 8, 1, eight + "<true>"), (122, 79, 40, 32, 8, 1, four + "<true>"),
        # long prefixes: passes of eight, of four, pipelined and general ones
        (300, 512, 104, 32, 8, 1, eight + "<true>"), (300, 512, 96, 32, 8, 1, four + "<true>"), (300, 1500, 128, 32, 8, 1, eight + "<true>"),
        (300, 1500, 96, 32, 8, 1, four + "<true>"), (250, 600, 128, 32, 32, 1, four + "<true>"), (250, 600, 96, 32, 32, 1, "stream_pipelined<false>"),
        (250, 600, 72, 32, 8, 1, "stream_pipelined<false>"), (250, 300, 96, 32, 32, 1, "stream_pipelined<false>"), (70, 834, 133, 32, 8, 1, four + "<false>"), (181, 1750, 88, 32, 8, 1, "stream_pipelined<false>"),
        (300, 512, 40, 32, 8, 1, "stream_pipelined<false>"),
        (64, 464, 109, 32, 8, 1, eight + "<false>"), (50, 424, 148, 32, 8, 1, four + "<false>"), (12, 2018, 156, 32, 32, 1, "stream_pipelined<false>"),
        (34, 1114, 111, 28, 4, 1, "stream_pipelined<false>"), (245, 676, 34, 32, 8, 1, "stream_pipelined<false>"),
        (43, 603, 113, 40, 40, 1, "stream_general"), (300, 700, 13, 32, 8, 1, "stream_general"), (512, 512, 29, 32, 32, 1, "stream_pipelined<true>"),
    ])


def test_calls_with_lengths(tmp_path):
    # packed<window steps, prefix tiles (resident; 3: three and more)>, and what is left to the kernels of calls without lengths
    check(tmp_path, "fwd", [
        (8, 1, 20, 4, 4, 1, "resident_packed<2,1>"), (8, 32, 20, 4, 4, 1, "resident_packed<2,1>"), (8, 33, 20, 4, 4, 1, "resident_packed<2,2>"),
        (8, 64, 24, 8, 2, 1, "resident_packed<1,2>"), (8, 65, 20, 4, 4, 1, "resident_packed<2,3>"), (40, 100, 20, 4, 4, 2, "resident_packed<2,3>"),
        (1024, 256, 25, 32, 8, 1, "resident_packed<1,3>"), (1024, 256, 26, 32, 8, 1, "resident_packed<2,3>"), (64, 256, 32, 32, 32, 1, "resident_packed<2,3>"),
        (64, 0, 20, 4, 4, 1, "resident_general"), (64, 256, 33, 32, 32, 1, "resident_general"),
        (300, 512, 20, 32, 8, 1, "stream_packed<1>"), (64, 257, 20, 32, 32, 1, "stream_packed<2>"), (700, 300, 33, 40, 40, 1, "stream_packed<2>"),
        (700, 300, 64, 40, 40, 1, "stream_packed<3>"), (65, 200, 64, 8, 8, 1, "stream_packed<3>"),
        # whole blocks of grouped heads, or one per candidate; longer suffixes; several prefixes
        (1500, 400, 32, 32, 8, 1, "stream_pipelined<true,true>"), (300, 700, 32, 40, 40, 1, "stream_pipelined<true,true>"),
        (300, 512, 40, 32, 8, 1, "stream_pipelined<false,true>"), (40, 300, 65, 40, 40, 1, "stream_general"), (40, 300, 20, 4, 4, 2, "stream_general"),
        (16, 128, 90, 32, 8, 1, "stream_candidate<false>"),
    ], lens=True)
    check(tmp_path, "bwd", [
        (1024, 256, 24, 32, 8, 1, "bwd_dq_packed<1>"), (500, 128, 20, 32, 32, 1, "bwd_dq_packed<2>"), (100, 0, 20, 4, 4, 1, "bwd_dq_packed<2>"),
        (500, 128, 64, 32, 32, 1, "bwd_dq_packed<2>"), (500, 128, 65, 32, 32, 1, "bwd_dq_resident"), (64, 257, 24, 32, 8, 1, "bwd_dq_mfma"),
        (512, 256, 32, 32, 8, 8, "bwd_dq_packed<2>"),
        (32, 128, 28, 32, 8, 1, "bwd_dq_unit"), (64, 256, 32, 32, 8, 1, "bwd_dq_unit"),     # few blocks, in full passes
    ], lens=True)
