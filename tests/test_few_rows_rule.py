"""Where few rows take one launch for the MLP, by what the workspace query asks for it (no GPU: nothing is launched)."""
import ctypes

import pytest

from paper_2306_06446_amd import binding as sa


def block_bytes(T, E, hid, moe):
    d = sa.SaBlockDesc()
    d.B, d.N, d.H, d.d, d.nbits, d.dv, d.hid, d.moe = 1, T, E // 64, 64, 64, 64, hid, int(moe)
    return sa.load_library().sa_block_workspace_bytes(ctypes.byref(d))


def partials(T, E):
    return (T + 15) // 16 * 4 * 16 * E * 4


# hidden layers of 8 E: a workgroup's chain is twice as long, and at E = 256 a CU has LDS for one of them
@pytest.mark.parametrize("last,E,hid,moe", [(112, 256, 2048, True), (416, 256, 1024, True), (1600, 64, 512, False), (1600, 128, 1024, False)])
def test_last_row_count(last, E, hid, moe):
    assert block_bytes(last, E, hid, moe) - block_bytes(last + 1, E, hid, moe) > partials(last, E) // 2


# Shift block of 64 columns: a hidden layer of 256 is one launch of its own in as little time
@pytest.mark.parametrize("T", [16, 784, 1600])
def test_narrow_hidden_layers_have_their_own_launch(T):
    assert block_bytes(T, 64, 512, False) - block_bytes(T, 64, 256, False) > partials(T, 64) // 2


# less than the query says is enough for other launches; less than those need is refused, with both sizes
def test_refused_workspaces_are_told_both_sizes():
    lib = sa.load_library()
    d = sa.SaBlockDesc()
    d.B, d.N, d.H, d.d, d.nbits, d.dv, d.hid, d.moe = 1, 197, 3, 64, 64, 64, 768, 1
    for n in ("q", "k", "v", "o", "workspace"):
        setattr(d, n, 0x1000)
    d.workspace_bytes = 16
    asked = lib.sa_block_workspace_bytes(ctypes.byref(d))
    assert lib.sa_block_forward(ctypes.byref(d), None) == -4
    text = lib.sa_last_error().decode()
    sizes = [int(w) for w in text.replace(",", "").split() if w.isdigit()]
    assert sizes[0] == asked and 16 < sizes[1] < asked and sizes[2] == 16, text
    d.workspace_bytes = sizes[1] - 1
    assert lib.sa_block_forward(ctypes.byref(d), None) == -4
    d.workspace_bytes = sizes[1]
    assert lib.sa_block_forward(ctypes.byref(d), None) == -1             # goes on to the next check: no weights are given
