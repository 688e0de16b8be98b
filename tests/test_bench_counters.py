"""bench.py quotes counter readings only of the kernels that it times: a reading names the digest of the sources it was taken with."""
import bench
from paper_1807_05358_amd import build

LINE = 'counters config=4 B=1024 traffic_bytes=2.0e+10 insts_valu=9.0e+09 {}kernel="k_loop_batch<false, false, 2, 64, 0, 4>"\n'


def test_readings_of_other_sources_are_not_quoted(tmp_path, monkeypatch):
    f = tmp_path / "counters.txt"
    monkeypatch.setattr(bench, "COUNTER_FILE", str(f))
    for label in ("", "sources=0123456789abcdef "):
        f.write_text("text\n" + LINE.format(label))
        assert bench.profiled_counters() == {}
    f.write_text(LINE.format(f"sources={build.kernel_digest()} "))
    assert bench.profiled_counters() == {4: {"kernel": "k_loop_batch<false, false, 2, 64, 0, 4>", "B": 1024, "traffic_bytes": 2.0e10, "insts_valu": 9.0e9}}


def test_the_digest_is_of_code_alone(tmp_path, monkeypatch):
    for name in build.KERNEL_UNITS + build.HEADERS:
        (tmp_path / name).write_text("int a; // one\n")
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    one = build.kernel_digest()
    (tmp_path / "ffsim_loop.h").write_text("int  a;\n/* two\nlines */\n")
    assert build.kernel_digest() == one
    (tmp_path / "ffsim_loop.h").write_text("int  b;\n")
    assert build.kernel_digest() != one
