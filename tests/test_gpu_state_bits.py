"""complex64 final states and shots keep their bits (needs an MI355X)."""

from __future__ import annotations

import json

import pytest

import state_cases
import workloads as W

torch = pytest.importorskip("torch")
import paper_2301_03251_amd as Q  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", list(state_cases.CASES))
def test_state_bits(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q.load()
    with open(state_cases.GOLDEN) as f:
        want = json.load(f)[name]
    assert state_cases.digests(name, Q, W, torch) == want
