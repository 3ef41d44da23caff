"""CPU checks of the benchmark's command line: one GPU only, and the workload list."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(*args):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args], capture_output=True,
                          text=True, timeout=300)


def test_more_than_one_gpu_is_refused():
    r = _run("--gpus", "2")
    assert r.returncode == 2
    assert "one GPU" in r.stderr or "1 GPU" in r.stderr or "single" in r.stderr


def test_unknown_workload_is_refused():
    r = _run("--workload", "no_such_surface")
    assert r.returncode == 2            # argparse: invalid choice
    assert "invalid choice" in r.stderr


def test_workloads_name_the_configs():
    sys.path.insert(0, ROOT)
    import bench
    import synth

    assert set(bench.WORKLOADS) == {"cap_2048", "sinusoid_4096", "sinusoid_128"}
    for name in bench.WORKLOADS:
        w = synth.config(name, side=16)
        assert w.name == name


def test_stored_fft_counters_are_of_the_current_engine(tmp_path, monkeypatch):
    """Counters taken on other code of the FFT passes, the kernels' or the engine's, are not
    reported; another wording of the comments does not matter."""
    sys.path.insert(0, ROOT)
    import bench

    names = [os.path.basename(p) for p in bench.FFT_SOURCES]
    assert sorted(names) == ["fft.hip", "fft_engine.h"]
    copies = []
    for p in bench.FFT_SOURCES:
        copies.append(tmp_path / os.path.basename(p))
        copies[-1].write_text(open(p, encoding="utf-8").read(), encoding="utf-8")
    monkeypatch.setattr(bench, "FFT_SOURCES", [str(p) for p in copies])
    summary = tmp_path / "summary.txt"
    summary.write_text(f"busy_pass1_fp32_valu: 0.5\nfft_code_sha256: {bench._code_sha(*bench.FFT_SOURCES)}\n")
    monkeypatch.setattr(bench, "PROFILE_FFT", str(summary))
    assert bench.stored_fft_busy() == {"pass1_fp32_valu": 0.5}
    for p in copies:
        text = p.read_text(encoding="utf-8")
        p.write_text("// a comment\n" + text, encoding="utf-8")
        assert bench.stored_fft_busy() == {"pass1_fp32_valu": 0.5}
        p.write_text(text + "\nint other;\n", encoding="utf-8")
        assert bench.stored_fft_busy() is None
        p.write_text(text, encoding="utf-8")
