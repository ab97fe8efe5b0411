"""What bench.py prints from committed measurements belongs to the sources it runs.  CPU only."""
import gc
import os
import types

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_committed_figures_are_used_only_for_the_sources_they_were_taken_of(tmp_path):
    table = "| kernel | calls | avg us |\n|---|---|---|\n| gram_density | 10 | 21.5 |\n"
    path = tmp_path / "t.md"
    for line, rows in ((f"Sources: {bench.source_digest()}", {"gram_density": ["10", "21.5"]}), ("Sources: 0123456789abcdef", {}), ("", {})):
        path.write_text(f"# a trace\n\n{line}\n\n{table}")
        assert {k: v for k, v in bench._profile_table("t.md", str(tmp_path)).items() if k != "kernel"} == rows
    assert bench._profile_table("absent.md", str(tmp_path)) == {}


def test_the_digest_is_of_the_headers_and_the_options_too(tmp_path, monkeypatch):
    from paper_2504_08966_amd import build
    files = [tmp_path / "paper_2504_08966_amd" / "csrc" / "a.hip", tmp_path / "include" / "a.h"]
    for f in files:
        f.parent.mkdir(parents=True)
        f.write_text("/* of several\n * lines */\nint f(int x);\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    seen = [bench.source_digest()]
    files[1].write_text("/* another */ int f(int x);\n")
    assert bench.source_digest() == seen[0]
    files[1].write_text("int f(int y);\n")
    seen.append(bench.source_digest())
    monkeypatch.setattr(build, "FLAGS", build.FLAGS + ["-O1"])
    seen.append(bench.source_digest())
    assert len(set(seen)) == 3


def test_the_digest_is_of_the_code(tmp_path):
    (tmp_path / "a.hip").write_text("int f(int x) {  // twice\n    return 2 * x;\n}\n")
    first = bench.source_digest(str(tmp_path))
    (tmp_path / "a.hip").write_text("// another comment\nint f(int x) { return 2 * x; }\n")
    assert bench.source_digest(str(tmp_path)) == first
    (tmp_path / "a.hip").write_text("int f(int x) { return 3 * x; }\n")
    assert bench.source_digest(str(tmp_path)) != first


def test_no_collection_while_calls_are_timed():
    torch = types.SimpleNamespace(cuda=types.SimpleNamespace(synchronize=lambda: None))
    kept, seen, at = [], [], []

    def collection(phase, info):
        seen.append(info["generation"])

    def call():
        at.append(len(seen))
        kept.extend([] for _ in range(20000))

    gc.callbacks.append(collection)
    try:
        bench.time_calls(torch, call, 10)
    finally:
        gc.callbacks.remove(collection)
    assert seen and at[0] == at[-1] and gc.isenabled()    # (one before the first call)
