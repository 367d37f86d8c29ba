"""Which kernels prompt attention takes on either side of the lines of the rule that decides whether the values are converted on the
way (one launch) or by a pass of their own (two), and how many workgroups the one launch has."""
import launch_log


def _launches(tmp_path, calls):
    return launch_log.run(tmp_path, f"""
        result = []
        for B, H, k, Tq, q_start, dense in {calls!r}:
            n = q_start + Tq
            tail = (128, 1, ctypes.c_float(0.1), P, P, N, None)
            if dense:
                st = L.chai_dense_prefill_attention(P, P, P, B, H, Tq, q_start, n, *tail)
            else:
                st = L.chai_prefill_attention(P, P, P, P, P, B, H, k, Tq, q_start, n, n, *tail)
            assert st == 0, (st, B, H, k, Tq, q_start, dense)
            result.append([[name, grid] for name, grid, block, lds, leave in launches()])
    """)


def _direct(got):
    assert len(got) == (1 if "prefill_direct" in got[0][0] else 2)
    return len(got) == 1


# (rows, heads, clusters, positions, behind): the last call that converts on the way, and one just past the line
_LINES = [
    ((15, 52, 8, 600, 512), (15, 52, 8, 600, 513)),       # five query tiles: many groups behind a long context
    ((14, 52, 8, 600, 4000), (15, 52, 8, 600, 4000)),
    ((20, 72, 8, 700, 128), (27, 52, 8, 700, 128)),       # six
    ((6, 52, 8, 700, 512), (6, 52, 8, 700, 513)),
    ((12, 52, 4, 860, 180), (12, 52, 4, 860, 181)),       # seven
    ((4, 32, 8, 872, 2000), (4, 32, 8, 872, 2090)),
    ((4, 52, 8, 1000, 66), (4, 52, 8, 1000, 67)),         # eight
]
_DENSE = [((4, 45, 860, 0), (4, 46, 860, 0))]             # seven


def test_both_sides_of_the_lines(tmp_path):
    calls = [c + (False,) for pair in _LINES for c in pair] + [(B, H, H, Tq, q, True) for pair in _DENSE for B, H, Tq, q in pair]
    for call, got in zip(calls, _launches(tmp_path, calls)):
        side = calls.index(call) % 2
        assert _direct(got) == (side == 0), (call, got)


def test_workgroups_of_small_calls(tmp_path):
    """A cluster of n heads is (n + 1) / 2 groups at most, (heads + clusters) / 2 a row: calls that are one round of the 256 CUs
    then have no workgroups beyond that, where the work list's bound would make it two."""
    calls = [(1, 72, 8, 646, 20, False), (1, 64, 24, 763, 4455, False), (2, 32, 8, 834, 3461, False), (1, 80, 2, 700, 3, False)]
    for (B, H, k, Tq, q, dense), got in zip(calls, _launches(tmp_path, calls)):
        most, tiles = B * min(H, (H + k) // 2), (Tq + 127) // 128
        assert got == [[got[0][0], (most + 7) // 8 * 8 * tiles]] and "prefill_direct" in got[0][0], got
