"""What the phase-stamp reader takes from the profiling build: workgroups of 128 or 256 rows, and per-wave loop stamps only where
the kernel writes them.  The library's debug entry point is replaced, so nothing here needs a GPU or that build."""
import types

import pytest

import paper_2505_20776_amd as sx
from paper_2505_20776_amd import phase_stamps


@pytest.mark.parametrize("rows,n_rows,waves,groups", [(256, 240, 8, 1), (128, 240, 4, 2), (128, 128, 4, 1), (256, 257, 8, 2)])
def test_workgroups(rows, n_rows, waves, groups):
    lib = types.SimpleNamespace(specext_debug_rows_per_workgroup=lambda desc: rows)
    desc = sx.make_desc(dtype=sx.SPECEXT_BF16, n_q_heads=32, n_kv_heads=8, head_dim=128, prefix_len=4096, n_tree=60)
    assert phase_stamps.workgroup_shape(lib, desc, n_rows) == (waves, groups)
    # 16 splits of the 60-node tree: 7.9 MB of spare partials, room for the loop stamps of eight-wave workgroups
    n = groups * 8 * 16
    assert phase_stamps.loop_stamps_written(waves, n, 16 * 32 * 60 * 128 * 2) == (waves == 8)
    assert not phase_stamps.loop_stamps_written(waves, n, (4 << 20) + n * waves * 320 - 1)
