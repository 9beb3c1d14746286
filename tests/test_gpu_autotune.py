"""The autotuner measures the path its tables are for: digit slices."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
dmp = pytest.importorskip("paper_2407_13299_amd")
from paper_2407_13299_amd import _lib, api, autotune  # noqa: E402


def test_measurements_run_on_digit_slices(monkeypatch):
    """Every run of S = 6, 7, 8 is given less than residue products need; sizes at
    which no accepted workspace is that small are left out."""
    lib = _lib.load()
    real, seen = api.purify, []

    def purify(h, nocc, **kw):
        s, kind = kw["slices"], kw.get("kind", "int8")
        if s != autotune.REF_SLICES:
            ws = kw["workspace"]
            n = h.shape[0]
            full = lib.dmp_purify_workspace_bytes(n, s, autotune.KIND_IDS[kind])
            assert ws.numel() < full if 6 <= s <= 8 else ws.numel() == full
            seen.append((n, s, kind))
        return real(h, nocc, **kw)
    monkeypatch.setattr(api, "purify", purify)
    quiet = lambda line: None
    rows = autotune.measure_tiles(sizes=(256, 1100), cases=(("int8", 7), ("int8", 5), ("fp16", 7)), rounds=1, log=quiet)
    assert {(k, s, n) for k, s, n, _ in rows} == {("int8", 7, 256), ("int8", 5, 256), ("int8", 5, 1100),
                                                 ("fp16", 7, 256), ("fp16", 7, 1100)}
    assert all(len(med) == 4 for _, _, _, med in rows)
    errors = autotune.measure(sizes=(128, 1100), slices=(5, 7), log=quiet)
    assert [(n, s) for n, s, _, _ in errors] == [(128, 5), (128, 7), (1100, 5)]
    assert (256, 7, "int8") in seen and (128, 7, "int8") in seen
