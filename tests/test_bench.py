"""What the benchmark reports from recorded profiles (no GPU calls)."""
import bench


def test_traffic_is_reported_for_its_launch_and_sources_alone(tmp_path, monkeypatch):
    f = tmp_path / "traffic.txt"
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(f))
    line = "# bench: kernel=sim traffic_bytes={} launch={} sources_sha256={}\n"
    f.write_text("# counters\n" + line.format(11, "grid=768,lds_blocks=128", bench.sources_sha256())
                 + line.format(12, "grid=768,lds_blocks=256", bench.sources_sha256())
                 + line.format(13, "grid=1024,lds_blocks=256", "0" * 64))
    assert bench.measured_traffic("grid=768,lds_blocks=128") == 11
    assert bench.measured_traffic("grid=768,lds_blocks=256") == 12
    assert bench.measured_traffic("grid=1024,lds_blocks=256") is None
    assert bench.measured_traffic("default") is None
    f.write_text("# bench: kernel=sim traffic_bytes=14 sources_sha256=" + bench.sources_sha256() + "\n")
    assert bench.measured_traffic("default") is None
