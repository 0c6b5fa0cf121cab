"""GPU tests of the autotuner's cache: a file of another set of kernel forms is measured
anew, and the partial round's lanes of a class with a fold form stay as set."""
import pytest

from paper_2111_11924_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = binding.Context(0)
    c.load_keys(inputs.make_keys([1024], 861))
    yield c
    c.close()


def test_cache_of_other_kernel_forms_is_not_applied(ctx, tmp_path):
    path = tmp_path / "tune.txt"
    ctx.autotune(str(path))
    first, *rows = path.read_text().splitlines()
    assert len(rows) == 1 and rows[0].split()[0] == "1024"
    stale = first.rsplit(" ", 1)[0]  # as before the forms were part of it
    path.write_text(f"{stale}\n1024 2 1 1 0.0\n")
    ctx.autotune(str(path))
    assert path.read_text().splitlines()[0] == first and ctx.window(1024) in (4, 5, 6)
    path.write_text(f"{first}\n1024 2 1 1 0.0\n")  # the same file under this signature is taken
    ctx.autotune(str(path))
    assert ctx.window(1024) == 2 and ctx.lanes(1024) == (1, 1)


def test_partial_round_setting_of_a_fold_class_stays(ctx, tmp_path):
    ctx.set_lanes(1024, 4, 2)
    ctx.autotune(str(tmp_path / "tune.txt"))
    assert ctx.lanes(1024)[1] == 2
