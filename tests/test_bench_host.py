"""Host-side parts of bench.py (no GPU): the recorded traffic of a kernel."""
import bench


def test_traffic_is_per_launch_of_the_measured_build(tmp_path, monkeypatch):
    f = tmp_path / "traffic.txt"
    src = bench.sources_hash("k_check_push")
    f.write_text("some text\n"
                 f"traffic kernel=k_check_push workload=rmat20 sources={src} per=step launches=1470 "
                 "fetch_bytes=1470000 write_bytes=294000\n"
                 "traffic kernel=k_check_push workload=rmat16 sources=0000000000000000 per=step launches=3 "
                 "fetch_bytes=1 write_bytes=1\n")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(f))
    tr = bench.measured_traffic("k_check_push", "rmat20")
    assert (tr["bytes"], tr["launches"], tr["bytes"] / tr["launches"]) == (1764000, 1470, 1200)
    assert bench.measured_traffic("k_check_push", "rmat16") is None  # taken from other sources


def test_recorded_traffic_names_its_launches():
    for line in open(bench.TRAFFIC_FILE):
        if line.startswith("traffic kernel=k_check_push"):
            assert " launches=" in line


def test_kernel_sources_exist():
    for kernel in bench.KERNEL_SOURCES:
        assert len(bench.sources_hash(kernel)) == 16
