"""What bench.py prints from committed measurements belongs to the sources it runs.  CPU only."""
import os

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_committed_figures_are_used_only_for_the_sources_they_were_taken_of(tmp_path):
    table = "| kernel | calls | avg us |\n|---|---|---|\n| gram_density | 10 | 21.5 |\n"
    path = tmp_path / "t.md"
    for line, rows in ((f"Sources: {bench.source_digest()}", {"gram_density": ["10", "21.5"]}), ("Sources: 0123456789abcdef", {}), ("", {})):
        path.write_text(f"# a trace\n\n{line}\n\n{table}")
        assert {k: v for k, v in bench._profile_table("t.md", str(tmp_path)).items() if k != "kernel"} == rows
    assert bench._profile_table("absent.md", str(tmp_path)) == {}


def test_the_digest_is_of_the_code(tmp_path):
    (tmp_path / "a.hip").write_text("int f(int x) {  // twice\n    return 2 * x;\n}\n")
    first = bench.source_digest(str(tmp_path))
    (tmp_path / "a.hip").write_text("// another comment\nint f(int x) { return 2 * x; }\n")
    assert bench.source_digest(str(tmp_path)) == first
    (tmp_path / "a.hip").write_text("int f(int x) { return 3 * x; }\n")
    assert bench.source_digest(str(tmp_path)) != first
