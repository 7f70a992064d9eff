"""GPU test of a tuning database written before the LU was among the choices of
the blocks' inversion: its entry is not taken, the choice is measured again
and kept in its place."""

import pytest

from gpu_common import product_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,prefix,gauss_jordan", [("fp64", "gj3:", (1, 6)), ("bf16", "gj3:f32:", (11, 16))])
def test_entry_from_before_the_lu_is_measured_again(precision, prefix, gauss_jordan, tmp_path):
    from paper_1709_05660_amd import MG
    p = product_problem("c0_2d_16x4")
    db, old = str(tmp_path / "new.db"), str(tmp_path / "old.db")
    mg = MG(p, precision=precision)
    assert mg.autotune(db) > 0
    mg.close()
    lines = open(db).read().split("\n")
    key = next(line.split()[0] for line in lines if line.startswith(prefix))
    before = ":".join(key.split(":")[:len(prefix.split(":")) + 2])
    with open(old, "w") as f:
        for line in lines:
            if line.startswith(prefix):
                f.write(f"{before} {gauss_jordan[1]}\n")
            elif line.startswith("gjg:"):
                f.write(":".join(line.split()[0].split(":")[:-1]) + f":{gauss_jordan[1]} {line.split()[1]}\n")
            elif line:
                f.write(line + "\n")
    mg = MG(p, precision=precision)
    assert mg.autotune(old) > 0
    assert mg.autotune(old) == 0
    mg.close()
    kept = dict(line.split() for line in open(old).read().split("\n") if line)
    print(precision, "old key", before, "entries", {k: v for k, v in kept.items() if k.startswith("gj")}, flush=True)
    assert key in kept and before not in kept
