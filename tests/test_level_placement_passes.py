"""Item memory placed by levels may be larger than in step order, but a pass of
few groups keeps them all."""
import json
import os

import pytest

import paper_1805_01450_amd as q
from workload import generate_circuit

PLANS = os.path.join(os.path.dirname(q.__file__), "plans")


@pytest.mark.parametrize("groups", [2, 5, 16])
def test_groups_per_pass_of_the_plain_placement(groups, monkeypatch):
    """7x7x30 in complex64 with a cap that just holds a number of groups as
    the program packs them."""
    with open(os.path.join(PLANS, "7x7x30.json")) as f:
        rec = json.load(f)
    cz = rec["circuit"]
    c = q.Circuit(generate_circuit(cz["n"], cz["depth"], cz["seed"]))

    def elems(**kw):
        return q.Plan(c, rec["sliced"], rec["order"], prec=q.QGM_C64, engine=q.QGM_ENGINE_WIDE, **kw).stats()["item_elems"]

    monkeypatch.setenv("QGM_WIDE_PREBUILT", "1")  # step order alone
    packed = elems()
    monkeypatch.delenv("QGM_WIDE_PREBUILT")
    cap = groups * packed * 64 * 8 + 4096
    assert cap // (elems(workspace_cap=cap) * 64 * 8) >= groups
