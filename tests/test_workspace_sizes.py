"""The workspace sizes that the library reports (host only)."""
import pytest


@pytest.fixture(scope="module")
def lib():
    import os
    from paper_1804_06926_amd import _lib
    if not os.path.exists(_lib.library_path()):
        from paper_1804_06926_amd import build
        build.build()
    return _lib


def test_least_workspace_never_falls_as_a_size_grows(lib):
    pairs = [0, 1, 1000, 90_000, 1 << 17, (1 << 17) + 1, 150_000, 1 << 22, 1 << 25, (1 << 31) - (1 << 20)]
    vertices = [0, 1, 100, 4096, 16_000, 16_384, 16_385, 20_000, 1 << 20, 1 << 27]
    for n0, n1 in zip(vertices, vertices[1:]):
        for E0, E1 in zip(pairs, pairs[1:]):
            assert lib._workspace_size_min(E0, n0) <= lib._workspace_size_min(E1, n0)
            assert lib._workspace_size_min(E0, n0) <= lib._workspace_size_min(E0, n1)
            assert lib._workspace_size_min(E0, n0) <= lib.workspace_size(E0, n0)
    assert lib._workspace_size_min(90_000, 16_000) < lib.workspace_size(150_000, 20_000) < lib.workspace_size(90_000, 16_000)
    for bad in ((-1, 5), (5, -1), ((1 << 31) - (1 << 19), 5)):
        with pytest.raises(lib.TCError):
            lib._workspace_size_min(*bad)
