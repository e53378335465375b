"""What a context's workspace holds beside the intensities: the gradient's and the m = 256 misfit's buffers are
bounded, whatever the number of patterns (host only)."""
import os

import pytest

E = pytest.importorskip("paper_2511_01793_amd.emagpie")

if not os.path.exists(E.LIB_PATH):
    pytest.skip("libemagpie.so not built", allow_module_level=True)

MIB = 1 << 20


def beside_the_data(m, n_pos, minibatch):
    c = E.Config(n_rows=1024, n_cols=1024, m=m, n_pos=n_pos, minibatch=minibatch, levels=1, alpha=0.01,
                 alpha_z=1.0, update_probe=1, joint_step=1, path=E.PATHS["graph"], seed=0)
    return E.workspace_size(c) - n_pos * m * m * 4


# 128 MiB of object slots, one probe slot per workgroup of the patch stage (1024, 512, 256; m = 256: 128
# patterns', and the stack buffer holds the object slots), 64 bytes per pattern of positions, orders and terms
@pytest.mark.parametrize("m, probe_mib", [(32, 16), (64, 32), (128, 32), (256, 64)])
@pytest.mark.parametrize("n_pos", [1, 100, 961, 4096, 8192, 20000])
def test_bounded_beside_the_data(m, probe_mib, n_pos):
    minibatch = min(32, n_pos)
    step = minibatch * m * m * 32  # numerators and stack of a minibatch, at most
    terms = n_pos * (64 + (16 * 8 if m == 256 else 0))
    assert beside_the_data(m, n_pos, minibatch) <= (128 + probe_mib + 1) * MIB + step + terms
