"""The default rates behind select_iters (no GPU)."""
import pytest

import scgen

P = pytest.importorskip("paper_2509_21037_amd")


@pytest.mark.parametrize("precision,low,high", [("fp64", 140, 175), ("mixed", 30, 40)])
def test_default_rates_match_the_measured_break_even(precision, low, high):
    """A 20^3 elasticity subdomain, glued face by face, in etree blocks: a batch
    of 64 breaks even after 146 to 167 applications in FP64 and 33 to 37 in
    mixed precision (two cards; assembly 173.7 and 181.1 ms, 85 and 89 mixed,
    explicit apply 2.87 ms, 1.54 mixed, implicit 4.08 and 3.94)."""
    s = scgen.box_subdomain("elasticity", (20, 20, 20), 1.0 / 20, 1, gluing="per_face")
    r = P.host_analyze(s, values=False, precision=precision, block_split="etree")
    assert low <= r["n_star"] <= high
