"""Workspace queries never ask for less when there is more to do, so that one
workspace sized for the largest input serves the smaller ones, across the sizes
where the parser's and the record writer's tiles change."""
import pytest

from paper_1607_06618_amd import gerbil as g


def around(*sizes):
    return sorted({max(0, s + d) for s in sizes for d in (-1, 0, 1)})


@pytest.mark.parametrize("lines", [0, 1000])
def test_parse_workspace_grows(lines):
    need = [g.gerbil_parse_workspace(n, min(n, lines)) for n in around(lines, 1 << 14, 1 << 16, 1 << 20, 1 << 27, 1 << 29, 1 << 31)
            if n >= lines]
    assert need == sorted(need)


def test_records_workspace_grows():
    need = [g.gerbil_records_workspace(n) for n in around(0, 1 << 10, 1 << 13, 1 << 21, 1 << 23, 1 << 24, 1 << 29)]
    assert need == sorted(need)
