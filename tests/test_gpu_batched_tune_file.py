"""The batched autotuner's cache file: an entry that an older library wrote (no kernel generation in its key) was
timed on other kernels, so it is not used, and the batch is tuned anew beside it."""
import json

import pytest

pytestmark = pytest.mark.gpu


def test_old_entry_is_not_used(tmp_path, monkeypatch):
    import torch
    from paper_2402_17913_amd import binding as B
    path = tmp_path / "tune.json"
    monkeypatch.setenv("NEUPHYS_TUNE_CACHE", str(path))
    sizes = [128, 64, 256]
    g = torch.Generator(device="cuda").manual_seed(0)
    f = [torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g) for n in sizes]

    def solve():
        x = [torch.zeros_like(t) for t in f]
        B.np_release_all()  # drops the process's settings, so that the file is read
        B.mg_poisson_solve_batched(f, x, [1.0 / n for n in sizes], smooth_prec=B.FP32, inner_cycles=0)
        return B.np_last_batched_settings()["source"]

    print("batched tune file", flush=True)
    assert solve() == "tuned"
    (key, entry), = json.load(open(path))["entries"].items()
    old = key.replace("|gen2|", "|")
    assert old != key

    def write(k, e):
        path.write_text('{"neuphys_batched_autotune": 1, "entries": {\n"%s": {"inner": %d, "nu": %d, "rm": %d, '
                        '"wg": %d, "ms": %.4f}\n}}\n' % (k, e["inner"], e["nu"], e["rm"], e["wg"], e["ms"]))

    write(key, entry)
    assert solve() == "file cache"
    write(old, dict(entry, rm=0))
    assert solve() == "tuned"
    assert {old, key} == set(json.load(open(path))["entries"])
