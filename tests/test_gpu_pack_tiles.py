"""Packing at the edges of its tiles (64 rows x 16 chunks, 64 rows x 64 row-scale groups), bit-exact."""
import pytest

from conftest import gpu_available
from synth import LayerSpec, paper_config
from test_gpu_parity import test_pack_sections_bit_exact as check_sections

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not gpu_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("spec", [
    LayerSpec("groups_71", M=65, N=9001, Kb=1, Ks=1, mu=8, S=300, g_r=128, g_s=128, seed=101),   # 72 + 3 chunks
    LayerSpec("one_group", M=130, N=1999, Kb=3, Ks=2, mu=4, S=129, g_r=1999, g_s=129, seed=102),  # 48 + 4 chunks
    LayerSpec("salient_tile", M=63, N=2048, Kb=1, Ks=1, mu=8, S=2048, g_r=256, g_s=2048, seed=103),  # 16 + 16 chunks
    LayerSpec("fine_global", M=70, N=2100, Kb=1, Ks=1, mu=4, S=40, g_r=32, g_s=40, seed=104),     # 17 + separator + 1
    paper_config("s16_tiles", 200, 2176, 1, 16, 128, seed=105)] +
    # every rotation within the row-scale groups of a chunk: groups of 8 to 64 columns at both mu, on the global side and
    # (with as many salient columns as give a ragged last chunk) the salient one
    [LayerSpec(f"groups_mu{mu}_{g}", M=67, N=300, Kb=2, Ks=1, mu=mu, S=150, g_r=g, g_s=g, seed=106)
     for mu in (4, 8) for g in (8, 16, 32, 64)], ids=lambda s: s.name)
def test_pack_tile_edges(spec):
    check_sections(spec)
