"""The tile table and steps on quad rows: their tiles, and the form of their
products, do not depend on the table, and the tuner spends nothing on them."""
import glob
import json
import os
from types import SimpleNamespace

import paper_1805_01450_amd as q
from workload import generate_circuit

PLANS = os.path.join(os.path.dirname(q.__file__), "plans")


def _circuit():
    with open(os.path.join(PLANS, "8x8x40.json")) as f:
        rec = json.load(f)
    cz = rec["circuit"]
    return q.Circuit(generate_circuit(cz["n"], cz["depth"], cz["seed"])), rec["sliced"], rec["order"]


def test_table_and_tuner_leave_quad_rows_alone(tmp_path, monkeypatch):
    """Every matrix-core step of the 8x8x40 plan is on quad rows.  A table that
    names a 16-item form and an odd ring for their shapes changes nothing in
    the generated kernels; tuning the plan needs no device and tunes no shape,
    and the entries of a table survive it."""
    c, sliced, order = _circuit()
    table = tmp_path / "tiles.txt"
    shapes = [(7, 7, 7), (6, 12, 7), (5, 10, 6), (8, 9, 6), (9, 6, 7)]
    table.write_text("".join(f"1 {i} {j} {k} 1 32768 0 {lay}\n" for (i, j, k), lay in zip(shapes, (1, 7, 48, 20, 2))))
    sources = []
    for path in (None, str(table)):
        out = tmp_path / f"dump{len(sources)}"
        out.mkdir()
        monkeypatch.setenv("QGM_DUMP_DIR", str(out))
        p = q.Plan(c, sliced, order, prec=q.QGM_C64, engine=q.QGM_ENGINE_WIDE, tile_table_path=path)
        (name,) = glob.glob(str(out / "qgm_wide_*.hip"))
        sources.append(open(name).read())
    assert all(f"i {i} j {j} k {k} fp32" in sources[0] for i, j, k in shapes)
    assert sources[0] == sources[1]
    assert q.qgm_plan_tune_tiles(p.h, str(table), SimpleNamespace(cuda_stream=0)) == 0
    kept = [line for line in table.read_text().splitlines() if not line.startswith("#")]
    assert len(kept) == len(shapes)
