"""The autotuner offers the variants that a configuration's kernels have, and no others."""
import pytest

from helpers import say
from paper_2312_09763_amd import matvis as mv
from paper_2312_09763_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n_ant", [("fp32", 66), ("fp32", 80), ("fp32", 96), ("bf16x3", 66), ("bf16x3", 96)])
def test_no_forming_split_without_a_full_block(tmp_path, precision, n_ant):
    # a variant that changes nothing may look faster by chance: it is not timed
    wl = synth.workload(2, n_ant=n_ant, n_src=500, n_time=2, n_freq=1)
    tuned, ms = mv.autotune(mv.config_for(wl, precision), **mv.device_inputs(wl, precision),
                            cache_path=str(tmp_path / "t.json"))
    say(f"autotune {precision}, {n_ant} antennas: tile={tuned.tile} ksplit={tuned.ksplit} {ms:.3f} ms")
    assert tuned.tile == 0 and ms > 0
