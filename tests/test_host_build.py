"""The build reads what the compiler says, however much that is."""
import importlib.util
import os
import stat

import pytest

import paper_2103_03936_amd


@pytest.mark.timeout(60)
def test_compiler_that_says_much(tmp_path, monkeypatch):
    spec = importlib.util.spec_from_file_location("pf_build_test", os.path.join(os.path.dirname(paper_2103_03936_amd.__file__), "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    fake = tmp_path / "hipcc"
    fake.write_text('#!/bin/sh\nhead -c 300000 /dev/zero | tr "\\0" "w"\nwhile [ $# -gt 1 ]; do [ "$1" = -o ] && : > "$2"; shift; done\n')
    fake.chmod(fake.stat().st_mode | stat.S_IXUSR)
    src = tmp_path / "csrc"
    src.mkdir()
    for n in range(3):
        (src / f"a{n}.hip").write_text("")
    monkeypatch.setenv("HIPCC", str(fake))
    monkeypatch.setattr(b, "HERE", str(tmp_path))
    monkeypatch.setattr(b, "CSRC", str(src))
    monkeypatch.setattr(b, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(b, "build_binding", lambda: None)
    b.build(jobs=1)
    assert sorted(p.name for p in (tmp_path / "_build").iterdir()) == ["a0.hip.o", "a1.hip.o", "a2.hip.o"]
