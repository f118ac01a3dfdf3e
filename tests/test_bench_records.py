"""bench.py prints the counter traffic of the kernels that it runs, or none."""
import bench


def _write(tmp_path, digest):
    (tmp_path / "profiles").mkdir(exist_ok=True)
    lines = ([f"Kernel sources: {digest} (bench.kernel_sources_digest)"] if digest else []) + ["MFMA convolution kernels, bytes per step: 123"]
    (tmp_path / "profiles" / "w_hbm_traffic.txt").write_text("\n".join(lines) + "\n")


def test_traffic_of_other_kernels_is_not_reported(tmp_path, monkeypatch):
    digest = bench.kernel_sources_digest()
    monkeypatch.setattr(bench, "kernel_sources_digest", lambda: digest)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_traffic("w") is None                # no profile
    _write(tmp_path, None)
    assert bench.measured_traffic("w") is None                # a profile that does not say of what
    _write(tmp_path, "0" * 16)
    assert bench.measured_traffic("w") is None                # of other kernels
    _write(tmp_path, digest)
    assert bench.measured_traffic("w") == 123


def test_digest_ignores_comments_and_follows_code(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2605_28657_amd" / "csrc"
    csrc.mkdir(parents=True)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    digests = []
    for text in ("int a = 1;  // one\n", "int a = 1; /* two\n lines */", "int a = 2;"):
        (csrc / "k.hip").write_text(text)
        digests.append(bench.kernel_sources_digest())
    assert digests[0] == digests[1] != digests[2]
