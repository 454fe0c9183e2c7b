"""The hash that ties recorded HBM traffic to the sources it was measured on follows the
code of the kernel and of its launch plan, and nothing else: an edit of a comment keeps
the figures, an edit of code, on the host side too, drops them."""
import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.fixture()
def copy(tmp_path, monkeypatch):
    for rel in bench.KERNEL_SOURCES:
        os.makedirs(os.path.dirname(str(tmp_path / rel)), exist_ok=True)
        shutil.copy(os.path.join(ROOT, rel), str(tmp_path / rel))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return tmp_path


def _edit(path, old, new):
    text = path.read_text()
    assert old in text
    path.write_text(text.replace(old, new, 1))


def test_comments_do_not_change_the_hash(copy):
    before = bench.sources_hash()
    for rel in bench.KERNEL_SOURCES:
        path = copy / rel
        path.write_text("// a new line\n" + path.read_text() + "\n/* and\n a block */\n")
    _edit(copy / bench.KERNEL_SOURCES[0], "template <int ROWS> struct Tile {", "template <int ROWS> struct Tile {  // tile")
    assert bench.sources_hash() == before


@pytest.mark.parametrize("rel,old,new", [
    (bench.KERNEL_SOURCES[0], "1.0f / 36.0f", "1.0f / 35.0f"),
    (bench.KERNEL_SOURCES[1], "kPhiFrac = 30", "kPhiFrac = 29"),
    (bench.KERNEL_SOURCES[2], "kMaxChunk = 128", "kMaxChunk = 64"),
])
def test_code_changes_the_hash(copy, rel, old, new):
    before = bench.sources_hash()
    _edit(copy / rel, old, new)
    assert bench.sources_hash() != before
