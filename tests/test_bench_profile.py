"""The traffic figures that bench.py reads from a committed profile are those of
the code that is measured."""
import os
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join("paper_2407_13299_amd", "csrc")


@pytest.fixture
def bench(tmp_path, monkeypatch):
    import importlib.util
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    shutil.copytree(os.path.join(ROOT, CSRC), tmp_path / CSRC)
    os.makedirs(tmp_path / "profiles")
    monkeypatch.setattr(mod, "ROOT", str(tmp_path))
    for s, name in ((7, "residue"), (5, "k_ozgemm")):
        with open(tmp_path / "profiles" / f"{name}_int8_s{s}_tb8192_traffic.md", "w") as f:
            f.write(f"code_sha256 = {mod.kernel_code_digest(mod.product_sources(s))}\nupdate_traffic_bytes = 5.0\n")
    return mod, tmp_path / CSRC


@pytest.mark.parametrize("file,old,new,stale", [
    ("modular.hpp", "kModCount[3] = {11, 13, 15}", "kModCount[3] = {11, 14, 15}", (7,)),
    ("residues.hpp", "struct ModSplits", "struct ModSplitz", (7,)),
    ("modular.hip", "NBUF - 1", "NBUF - 2", (7,)),
    ("ozgemm.hip", "__launch_bounds__(128 * RB", "__launch_bounds__(64 * RB", (5,)),
    ("ldsload.hpp", "buffer_load_dwordx4", "buffer_load_dword", (7, 5)),
    ("layout.hpp", "kTileM = 128", "kTileM = 64", (7, 5)),
    ("plan.cpp", "G = 1024 / edge", "G = 512 / edge", (7, 5)),
    ("modular.hip", "// Residue products", "// Other words", ())])
def test_a_change_of_the_products_voids_the_figures(bench, file, old, new, stale):
    mod, csrc = bench
    assert [mod.profiled_traffic("int8", s) for s in (7, 5)] == [5.0, 5.0]
    text = (csrc / file).read_text()
    assert old in text
    (csrc / file).write_text(text.replace(old, new))
    for s in (7, 5):
        assert mod.profiled_traffic("int8", s) == (None if s in stale else 5.0)
