"""The shipped network's plan biases come out of the committed rows: fitted to
the instances of even number, judged on the others (no GPU; the times are the
measured ones in planner_rows.npz)."""
import json

import numpy as np

from oracle import mlp_ref
from paper_1905_13376_amd import learned as M


def test_shipped_weights_are_the_refit(tmp_path):
    w, rep = M.refit()
    np.testing.assert_array_equal(w, np.load(M.WEIGHTS, allow_pickle=False))
    assert rep == json.load(open(M.REPORT))
    # again from weights whose plan biases are others: the report holds the trained ones
    v = w.copy()
    v[M.P - M.OUT + 2: M.P - M.OUT + 8] += 3
    other = tmp_path / "w.npy"
    np.save(other, v)
    np.testing.assert_array_equal(M.refit(weights=str(other))[0], w)


def test_held_out_half_beats_the_analytic_planner():
    w, D = np.load(M.WEIGHTS, allow_pickle=False), M.load_rows([M.ROWS])
    assert len(D["kind"]) == 400 and D["counts_exact"].all()
    odd = {k: v[1::2] for k, v in D.items()}
    r = M.score(M.predict_host(w, odd["features"]), odd)
    assert r["learned"] < r["analytic"] < r["always_3way"]
    held = json.load(open(M.REPORT))["plan_bias_refit"]["held_out"]
    assert held["learned"] == r["learned"] and held["analytic"] == r["analytic"]


def test_the_fit_uses_only_its_rows():
    """Other times of the odd rows leave the fit as it is."""
    w, D = np.load(M.WEIGHTS, allow_pickle=False), M.load_rows([M.ROWS])
    Y = M.predict_host(w, D["features"])
    even = {k: v[0::2] for k, v in D.items()}
    a = M.refit_plan_bias(Y[0::2], even)
    D["times"][1::2] *= 7.0
    np.testing.assert_array_equal(M.refit_plan_bias(Y[0::2], {k: v[0::2] for k, v in D.items()}), a)
    # no constant in the grid does better one logit at a time
    own = M.score(Y[0::2] + np.concatenate([[0, 0], a, [0, 0, 0]]), even)["learned"]
    for k in (1, 2, 4, 5):
        for g in (-8.0, -1.0, 1.0, 8.0):
            b = a.copy()
            b[k] += g
            assert M.score(Y[0::2] + np.concatenate([[0, 0], b, [0, 0, 0]]), even)["learned"] >= own - 1e-9


def test_host_outputs_equal_the_reference():
    w = np.load(M.WEIGHTS, allow_pickle=False)
    p, o = {}, 0
    for name, shape in M.SHAPES:
        k = int(np.prod(shape))
        x = w[o:o + k].reshape(shape)
        p[name] = mlp_ref.bf16_round(x) if name.startswith("W") else x
        o += k
    X = M.load_rows([M.ROWS])["features"][:40]
    np.testing.assert_allclose(M.predict_host(w, X), mlp_ref.forward(p, X)[0], rtol=1e-9, atol=1e-9)
