"""The library's kernel choice and KV-cache plan (host code, asked through the
probe library; no GPU needed), on 256 compute units unless said otherwise."""
import pytest

from tests.probes import route


@pytest.mark.parametrize("mode", ["fast", "fp8qk"])
def test_a_split_is_one_generation_of_workgroups(mode):
    # A split is planned as one workgroup per compute unit: no XCD (32 of them) may
    # get more, also where the tiles do not divide by 8
    seen = set()
    for heads in range(1, 130):
        for nk in (2100, 9000, 60000, 131001):
            for G, nq in ((4, 1), (1, 32), (1, 48)):
                r = route(heads, G, 1, nq, nk, 128, 128, mode=mode)
                if r["C"] > 1:
                    assert r["slots"] <= 32 and r["slots"] * 8 >= r["units"] * r["C"], (heads, nk, G, nq, r)
                    seen.add(r["units"])
    assert {1, 2, 3, 5, 9, 11, 12, 21, 33} <= seen
