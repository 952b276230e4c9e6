"""PSN_TUNE_CACHE records name tiles of the library that wrote them: a record
without a tag, or with another table's, is timed anew; one with this library's
tag is taken without timing."""
import pytest

from gpu_common import torch_cuda

pytestmark = pytest.mark.gpu
psn = pytest.importorskip("paper_1612_01799_amd")


def _records(path):
    return [line.split() for line in path.read_text().split("\n") if line.strip()]


@pytest.mark.parametrize("n,dtype,code", [(96, "f64", 0), (128, "f32", 1)])
def test_records_of_another_table_are_timed_anew(n, dtype, code, tmp_path, monkeypatch):
    torch_cuda()
    print(f"case n={n} {dtype}", flush=True)
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("PSN_TUNE_CACHE", str(path))
    build = lambda: psn.Plan(n, 2.0, 1e-12, dtype).build().info()["schedule"]
    path.write_text(f"{n} {code} 3 1\n")
    chosen = build()
    assert len(_records(path)) == 2
    last = _records(path)[-1]
    assert last[:4] == [str(n), str(code), str(chosen[0]), str(chosen[1])]
    tag = last[4]
    other = f"{int(tag, 16) ^ 1:08x}"
    path.write_text(f"{n} {code} 3 1 {other}\n")
    assert build() == chosen and len(_records(path)) == 2
    for want in ((1, 2), (3, 0)):   # this library's own: taken, nothing appended
        path.write_text(f"{n} {code} 0 0 {tag}\n{n} {code} {want[0]} {want[1]} {tag}\n{n} {code} 2 2\n")
        assert build() == want and len(_records(path)) == 3
