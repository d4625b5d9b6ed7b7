"""The shipped planner on instances that had no part in anything fitted: not
in the training (other seeds), not in the plan biases' fit (the instances of
odd number of the 400 whose even ones the biases were fitted to)."""
import pytest

pytestmark = pytest.mark.gpu


def test_shipped_planner_on_instances_without_a_part_in_the_fit():
    import paper_1905_13376_amd as mj
    from paper_1905_13376_amd import learned as M
    ctx = mj.Context()
    pl = M.use_shipped(ctx)
    rows = [M.label_instance(ctx, x) for x in M.planner_instances(400, 7_500_000, 3.0, 6.0)[1::2]]
    D = M.rows_to_arrays(rows)
    assert D["counts_exact"].all()
    r = M.evaluate(pl, D)
    print(r)
    assert r["instances"] == 200 and r["learned"] < r["analytic"]
    ctx.set_planner(None)
