"""The tuner's candidates hold every count of x lines that the built-in shapes
choose from. With ny = 54 lines of 16 pairs the powers of two leave blocks of 256
threads with 32 pairs at most; the built-in 6 lines have 96, in a third of the
blocks."""
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def test_counts_that_are_no_power_of_two(gpu, tmp_path, monkeypatch):
    monkeypatch.setenv("PSV_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    grid = gpu.Grid(32, 54, 512, 1.0, 1.0, 1.0)
    built_in, tuned = gpu.Plan(grid).get_shape(), gpu.Plan(grid, autotune=2).get_shape()
    say(f"built-in {built_in}, tuned {tuned}")
    assert tuned["lines_x"] in (3, 6) and tuned["lines_x_inv"] in (3, 6)


@pytest.mark.parametrize("nx,ny,nz", [(1024, 8, 6), (256, 64, 96)])
def test_choice_is_found_again(gpu, tmp_path, monkeypatch, nx, ny, nz):
    """A tuned shape that is the built-in one, with more LDS than the other
    candidates may take, is read back: the second plan does not tune again."""
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("PSV_AUTOTUNE_CACHE", str(cache))
    grid = gpu.Grid(nx, ny, nz, 1.0, 1.0, 1.0)
    first = gpu.Plan(grid, autotune=2).get_shape()
    second = gpu.Plan(grid, autotune=2).get_shape()
    say(f"{nx}x{ny}x{nz} {first}: {cache.read_text()}")
    assert second == first
    assert len([ln for ln in cache.read_text().splitlines() if f":{nx}x{ny}x{nz}:" in ln]) == 1
