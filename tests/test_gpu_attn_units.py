"""Attention work units at every GQA group: how a wave finds its rows (member
positions in the unit, scalar or per-lane reads of the member list), blocks
of a run's end that opened after the plan was made (in this launch, or in an
earlier step of the same plan), one- and two-tile units that wait for their
own append.  36 steps with no round between them cross two block openings of
every trace; every output against the oracle at the parity bar."""
import pytest

from _parity import replay
from workload import Workload, tiny

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("g", [1, 2, 4, 8, 16])
def test_groups_and_growing_runs(g, kv_dtype):
    cfg = tiny(kv_dtype=kv_dtype, n_q_heads=2 * g, gens=(2, 6, 24), prompt_len=37, seg_hi=90, steps=36, interval=40,
               keep=12, n_parents=12)
    replay(Workload(cfg), check_pool_every_step=True, quantise_on_append=kv_dtype != "bf16")
