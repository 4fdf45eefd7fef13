"""bench.py's roofline records name the kernels that ran: the stages for a
forward run without a tally in large chunks, the lane machine for the others;
and every name it looks for is a kernel of the built library."""
import re
import subprocess
import sys

import pytest

from conftest import ROOT
from paper_1410_1629_amd import binding as B

sys.path.insert(0, ROOT)
import bench  # noqa: E402

STATS = dict(x_path=10 ** 9, x_locate=10 ** 8, x_peel=4 * 10 ** 9, x_queue=4 * 10 ** 9, deposits=0, d_queue=0,
             peels=10 ** 7, life_ms=800.0, peel_ms=350.0, dep_ms=0.0, life_launches=4, packages=10 ** 8)


def _records(adjoint=False, tally=False, **st):
    return bench.rooflines(dict(STATS, **st), 1, adjoint, "clumpy", 1200.0, "level", tally=tally)


def test_a_large_run_without_a_tally_is_in_stages():
    r = _records()
    assert set(r) == {"stages_forward", "peel_tau_forward"}
    assert r["stages_forward"]["launches_per_step"] == 4 and r["stages_forward"]["launch_ms"] == 200.0
    for k in bench.STAGES:
        assert bench.KERNELS[k] in r["stages_forward"]["kernel"]
    assert "k_life" not in r["stages_forward"]["kernel"]


@pytest.mark.parametrize("case", [dict(tally=True), dict(packages=4 * bench.STAGE_ITEMS - 1)])
def test_other_forward_runs_are_the_lane_machines(case):
    r = _records(**case)
    assert set(r) == {"life_forward", "peel_tau_forward"} and "k_life<" in r["life_forward"]["kernel"]


def test_an_adjoint_with_a_tape_is_the_lane_machines():
    r = _records(adjoint=True, peel_ms=0.0, dep_ms=100.0, d_queue=4 * 10 ** 9)
    assert set(r) == {"life_adjoint", "peel_deposit"} and "k_life<" in r["life_adjoint"]["kernel"]


def test_an_adjoint_without_a_tape_replays_once_in_stages():
    r = _records(adjoint=True, dep_ms=100.0, d_queue=2 * 10 ** 9, life_launches=8)
    assert set(r) == {"stages_adjoint", "peel_tau_adjoint", "peel_deposit"}
    assert "k_leg" in r["stages_adjoint"]["kernel"] and bench.KERNELS["life_adjoint"] in r["stages_adjoint"]["kernel"]


def test_the_stages_bytes_are_those_of_all_their_kernels(tmp_path, monkeypatch):
    import json
    (tmp_path / "profiles").mkdir()
    w = {k: {"bytes_per_launch": 10.0 * (i + 1), "dispatches": 4 if k in ("emit", "tail") else 48}
         for i, k in enumerate(bench.STAGES)}
    (tmp_path / "profiles" / "traffic.json").write_text(json.dumps({"source_hash": "x", "workloads": {"clumpy": w}}))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "source_hash", lambda: "x")
    assert bench.traffic_for("clumpy", "stages_forward") == 10.0 + 60.0 + 12 * (20.0 + 30.0 + 40.0 + 50.0)
    del w["leg"]
    (tmp_path / "profiles" / "traffic.json").write_text(json.dumps({"source_hash": "x", "workloads": {"clumpy": w}}))
    assert bench.traffic_for("clumpy", "stages_forward") is None


def test_the_names_are_kernels_of_the_library():
    B.load()
    out = subprocess.run(["nm", "-C", B.LIB_PATH], check=True, capture_output=True, text=True).stdout
    stubs = {re.sub(r"^.*__device_stub__", "", ln) for ln in out.splitlines() if "__device_stub__" in ln}
    for key, name in bench.KERNELS.items():
        short = name.replace("void mcrt::", "").replace("mcrt::", "", 1) if name.startswith("mcrt::") else \
            name.replace("void mcrt::", "", 1)
        assert short in stubs, (key, short)
