"""Lines of an autotune cache that were timed on other step kernels are not taken:
the lattice is tuned again and its new choice is the one that holds."""

import json

import pytest

import parity as PT
from paper_1309_6726_amd import inputs
from test_gpu_parity import lbm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["moments", "populations"])
def test_lines_of_other_kernels_are_not_taken(lbm, tmp_path, monkeypatch, scheme):  # noqa: F811
    import torch
    path = tmp_path / "tune.jsonl"
    monkeypatch.setenv("LBM_AUTOTUNE_CACHE", str(path))
    prob = inputs.config0()
    PT.say(f"[tune cache] {scheme}")
    first = lbm.Sim.from_problem(prob, scheme=scheme)
    tile, _ = first.autotune(steps=2)
    key = json.loads(path.read_text())["key"]
    arch = torch.cuda.get_device_properties(0).gcnArchName.replace(":", "_")
    oldest = f"{arch}:256x32:0:{scheme[:3]}"  # before keys counted the kernels
    # 48 rows and 256 threads are no candidate for this lattice
    stale = {"tx": 256, "sy": 48, "ms": 0.001, "nt": 1}
    others = [oldest, key[:-1] + "1", key + "0"]
    path.write_text("".join(json.dumps({"key": k, **stale}) + "\n" for k in others))
    again = lbm.Sim.from_problem(prob, scheme=scheme)
    got, ms = again.autotune(steps=2)
    assert got[0] == 64 and got[1] != 48 and ms > 0.001
    lines = [json.loads(line) for line in path.read_text().splitlines()]
    assert len(lines) == 4 and lines[3]["key"] == key and (lines[3]["tx"], lines[3]["sy"]) == got
    # a line of these kernels is
    path.write_text(json.dumps({"key": key, **stale}) + "\n")
    cached = lbm.Sim.from_problem(prob, scheme=scheme)
    assert cached.autotune(steps=2)[0] == (256, 48) and cached.load_hint() == 1
    assert tile[0] == 64
