"""The work a user has this evaluator do, as a list of measurable cases.

A case is one evaluation call: a data set, a list of hyper-parameter suggestions and the entry point that is
called with them.  Data sets are the repository's synthetic stand-ins (inputs.py) at the sizes of its five
configurations and around them; suggestions are spread over the configurations' search boxes.  Widths and batch
sizes are the same for every seed (spread evenly over their ranges), so a case's work is a fixed number; the
data, folds, learning rates, penalties, initial weights and minibatch orders come from the seed.

Learning rates stop at 1e-3, the usual default: further up some runs amplify the last bit of a sum until their
scores say nothing about the arithmetic.  Epoch counts are cut so that a pass is short; every epoch is the same
work.

Fields of a case
  data         clusters | digits | regression | binary | mixture    generator of inputs.py
  rows, features, classes (0 regression, 1 one logit, >= 2 softmax)
  suggestions  how many; folds; epochs
  layers_lo/hi hidden layers (0 is a linear model), dealt round-robin; width_lo/hi, batch_lo/hi (0: full batch)
  solver       adam | sgd (Nesterov momentum)
  patience, val_fraction   early stopping on held-out training rows (0: off)
  bf16         inputs and operands in bfloat16
  entry        evaluate   suggestions as dicts, scores and status back (what the suggest-observe loop does)
               per_fold   the same with the scores of every fold
               planned    records and workspace kept by the caller
               driver     driver.gpu_evaluator: scores on the host
               static     the allocation-free entry point, outputs kept by the caller
               holdout    one model per suggestion, scored on the rows of no fold
"""
import math

import numpy as np
import torch

from paper_2012_04201_amd import binding, driver, inputs

_BASE = {"data": "binary", "rows": 569, "features": 30, "classes": 2, "suggestions": 8, "folds": 5, "epochs": 20,
         "layers_lo": 1, "layers_hi": 1, "width_lo": 50, "width_hi": 200, "batch_lo": 16, "batch_hi": 256,
         "solver": "adam", "patience": 0, "val_fraction": 0.0, "bf16": False, "entry": "evaluate"}


def _case(name, **fields):
    return dict(_BASE, name=name, **fields)


def listed():
    return [
        # Sequential search: one suggestion at a time on an iris-sized set, from a loop that must not allocate.
        _case("one_suggestion", data="clusters", rows=150, features=4, classes=3, suggestions=1, width_lo=20,
              width_hi=20, batch_lo=0, batch_hi=0, entry="static"),
        # One iteration of one study on the tiny classification configuration, scores back on the host.
        _case("tiny_study", data="clusters", rows=150, features=4, classes=3, width_lo=8, width_hi=32, batch_lo=0,
              batch_hi=0, entry="driver"),
        # One iteration of one study on the digits-shaped configuration: 40 models, few for the chip.
        _case("digits_study", data="digits", rows=1797, features=64, classes=10, epochs=10),
        # One iteration of one study on the regression configuration: SGD with Nesterov momentum, fold scores asked for.
        _case("regression_study", data="regression", rows=506, features=13, classes=0, batch_hi=128, epochs=30,
              solver="sgd", entry="per_fold"),
        # One iteration of 256 studies at once: the many-studies configuration, thousands of small models.
        _case("many_studies", suggestions=2048),
        # The same for models without a hidden layer (linear / logistic regression), the cheapest of the space.
        _case("many_linear", suggestions=2048, layers_lo=0, layers_hi=0),
        # 64 studies of the digits shape: the chip full of the wider single-layer models.
        _case("many_digits", data="digits", rows=1797, features=64, classes=10, suggestions=512, epochs=5),
        # Early stopping on a validation fraction with a one-logit head: the option the tuned models use most.
        _case("early_stopping", classes=1, suggestions=512, patience=3, val_fraction=0.1),
        # Depth is part of the search: one to three hidden layers in fp32, 32 studies in one call.
        _case("depth_search", suggestions=256, layers_lo=1, layers_hi=3, width_lo=16, width_hi=128, epochs=10),
        # A real set down-sampled to 10,000 rows, one study, ragged feature count.
        _case("rows_10k", rows=10000, features=45, epochs=3),
        # The scale-up configuration in bfloat16: two wide hidden layers on 20,000 rows, 32 studies in one call.
        _case("scale_up", data="mixture", rows=20000, features=128, classes=10, suggestions=256, epochs=6, layers_lo=2,
              layers_hi=2, width_lo=128, width_hi=256, batch_lo=256, batch_hi=256, bf16=True, entry="planned"),
        # Generalization score of every study's best suggestion: one model each, trained on the rows of all folds.
        _case("holdout_bf16", data="mixture", rows=10000, features=128, classes=10, suggestions=64, epochs=6,
              layers_lo=1, layers_hi=2, width_lo=128, width_hi=256, batch_lo=64, batch_hi=256, bf16=True,
              entry="holdout"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# What the listed cases stand for: per kind the ranges its sizes are drawn from.
def _one(rng):
    return dict(data="clusters", rows=_log(rng, 60, 400), features=rng.randint(3, 15), classes=rng.randint(2, 4),
                suggestions=rng.randint(1, 4), width_lo=8, width_hi=rng.randint(9, 40), batch_lo=0, batch_hi=0,
                entry="static")


def _tiny(rng):
    return dict(data="clusters", rows=_log(rng, 60, 400), features=rng.randint(3, 15), classes=rng.randint(2, 4),
                suggestions=rng.randint(6, 12), folds=rng.randint(3, 6), width_lo=8, width_hi=rng.randint(20, 40),
                batch_lo=0, batch_hi=0, entry=rng.choice(["driver", "evaluate"]))


def _digits(rng):
    return dict(data="digits", rows=_log(rng, 600, 2400), features=rng.randint(40, 80), classes=rng.randint(5, 12),
                suggestions=rng.randint(6, 12), width_hi=rng.randint(120, 200), epochs=rng.randint(4, 9))


def _regression(rng):
    return dict(data="regression", rows=_log(rng, 250, 1500), features=rng.randint(8, 29), classes=0, batch_hi=128,
                suggestions=rng.randint(6, 12), width_hi=rng.randint(120, 200), epochs=rng.randint(10, 20),
                solver=rng.choice(["sgd", "adam"]), entry="per_fold")


def _studies(rng):
    return dict(rows=_log(rng, 300, 900), features=rng.randint(14, 31), suggestions=_log(rng, 256, 1600),
                batch_hi=rng.randint(100, 256), width_hi=rng.randint(120, 200), epochs=rng.randint(5, 12),
                folds=rng.randint(3, 6))


def _linear(rng):
    return dict(rows=_log(rng, 300, 900), features=rng.randint(8, 60), suggestions=_log(rng, 256, 2048),
                batch_hi=rng.randint(100, 256), layers_lo=0, layers_hi=0, epochs=rng.randint(5, 20))


def _wide(rng):
    return dict(data="digits", rows=_log(rng, 600, 2000), features=rng.randint(40, 80), classes=rng.randint(5, 12),
                suggestions=_log(rng, 64, 400), width_hi=rng.randint(120, 200), epochs=rng.randint(2, 5))


def _stopping(rng):
    return dict(rows=_log(rng, 300, 900), features=rng.randint(8, 31), classes=1, suggestions=_log(rng, 64, 512),
                width_hi=rng.randint(120, 200), patience=rng.randint(2, 5), val_fraction=rng.choice([0.1, 0.15, 0.2]),
                epochs=rng.randint(8, 16))


def _depth(rng):
    return dict(rows=_log(rng, 300, 900), features=rng.randint(8, 60), suggestions=_log(rng, 24, 256),
                layers_lo=rng.randint(1, 2), layers_hi=3, width_lo=16, width_hi=rng.randint(64, 128),
                epochs=rng.randint(4, 8))


def _rows(rng):
    return dict(rows=_log(rng, 4500, 10000), features=rng.randint(20, 60), suggestions=rng.randint(6, 12),
                width_hi=rng.randint(120, 200), epochs=rng.randint(1, 3))


def _scale(rng):
    return dict(data="mixture", rows=_log(rng, 5000, 20000), features=8 * rng.randint(8, 16),
                classes=rng.randint(2, 12), suggestions=_log(rng, 48, 160), epochs=rng.randint(2, 5),
                layers_lo=rng.randint(1, 2), layers_hi=2, width_lo=128, width_hi=rng.randint(200, 256), batch_lo=256,
                batch_hi=256, bf16=True, entry="planned")


def _holdout(rng):
    return dict(data="mixture", rows=_log(rng, 3000, 10000), features=8 * rng.randint(8, 16),
                classes=rng.randint(2, 12), suggestions=_log(rng, 16, 96), epochs=rng.randint(2, 6), layers_lo=1,
                layers_hi=2, width_lo=128, width_hi=rng.randint(200, 256), batch_lo=64, batch_hi=256, bf16=True,
                entry="holdout")


_KINDS = [_one, _tiny, _digits, _regression, _studies, _linear, _wide, _stopping, _depth, _rows, _scale, _holdout]


def draw(rng):
    return dict(_BASE, **rng.choice(_KINDS)(rng))


def _spread(i, lo, hi, step):
    """The i-th of a sequence of whole numbers spread evenly over [lo, hi] (multiples of an irrational, modulo 1)."""
    return lo + int((i + 0.5) * step % 1.0 * (hi - lo + 1))


def _shapes(case):
    """(hidden widths, batch size) of every suggestion."""
    out = []
    for b in range(case["suggestions"]):
        depth = case["layers_lo"] + b % (case["layers_hi"] - case["layers_lo"] + 1)
        hidden = [_spread(3 * b + l, case["width_lo"], case["width_hi"], 0.6180339887498949) for l in range(depth)]
        out.append((hidden, _spread(b, case["batch_lo"], case["batch_hi"], 0.4142135623730950)))
    return out


def _suggestions(case, rng):
    def logu(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    sgd = case["solver"] == "sgd"
    hps = []
    for hidden, batch in _shapes(case):
        h = {"hidden": hidden, "solver": case["solver"], "nesterov": sgd, "batch_size": batch,
             "epochs": case["epochs"], "lr": logu(1e-4, 1e-3), "alpha": logu(1e-5, 1.0),
             "momentum": logu(0.5, 0.95) if sgd else 0.9, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8,
             "seed": int(rng.integers(0, 2 ** 63 - 1))}
        if case["patience"]:
            h.update(tol=1e-4, n_iter_no_change=case["patience"], validation_fraction=case["val_fraction"])
        hps.append(h)
    return hps


def _data(case, seed):
    n, d, c = case["rows"], case["features"], case["classes"]
    if case["data"] == "clusters":
        return inputs.data_clusters(seed, n=n, d=d, n_classes=c)
    if case["data"] == "digits":
        return inputs.data_digits(seed, n=n, d=d, n_classes=c)
    if case["data"] == "regression":
        return inputs.data_regression(seed, n=n, d=d)
    if case["data"] == "binary":
        return inputs.data_binary(seed, n=n, d=d)
    return inputs.data_mixture(seed, n=n, d=d, n_classes=c)


def prepare(case, seed):
    seeds = np.random.SeedSequence(seed).generate_state(3)
    X, y = _data(case, int(seeds[0]))
    fold = inputs.make_folds(case["rows"], case["folds"], int(seeds[1]))
    if case["entry"] == "holdout":  # one part in `folds` of the rows is in no fold
        fold = np.where(fold == 0, -1, fold - 1).astype(np.int32)
    cfg = {"X": X, "y": y, "n_classes": case["classes"], "dtype": binding.BF16 if case["bf16"] else binding.F32,
           "fold_idx": fold, "n_folds": case["folds"]}
    hps = _suggestions(case, np.random.default_rng(int(seeds[2])))
    device = torch.device("cuda:0")
    state = {"entry": case["entry"], "hps": hps}
    if case["entry"] == "driver":
        state["evaluate"] = driver.gpu_evaluator(cfg)
        return state
    X, y, fold = binding.to_device(cfg, device)
    state.update(X=X, y=y, fold=fold, classes=case["classes"], folds=case["folds"], dtype=cfg["dtype"])
    if case["entry"] == "planned":
        state["records"] = binding.make_hparams(hps)
        need = binding.bbo_mlp_workspace_bytes(case["rows"], case["features"], case["classes"], case["folds"], hps,
                                               cfg["dtype"], state["records"])
        state["workspace"] = binding.alloc_workspace(need, device)
    if case["entry"] == "static":
        state["scores"] = torch.empty(len(hps), 2, dtype=torch.float32, device=device)
        state["status"] = torch.empty(len(hps), dtype=torch.int32, device=device)
    return state


def run(state):
    s, entry = state, state["entry"]
    if entry == "driver":
        return s["evaluate"](s["hps"])
    if entry == "holdout":
        return binding.bbo_mlp_holdout_eval(s["X"], s["y"], s["classes"], s["fold"], s["hps"], s["dtype"])
    args = (s["X"], s["y"], s["classes"], s["fold"], s["folds"], s["hps"], s["dtype"])
    if entry == "static":
        return binding.bbo_mlp_cv_eval_static(*args, scores=s["scores"], status=s["status"])
    if entry == "planned":
        return binding.bbo_mlp_cv_eval(*args, workspace=s["workspace"], hp_arr=s["records"])
    return binding.bbo_mlp_cv_eval(*args, want_per_fold=entry == "per_fold")


def work(case):
    """Multiply-adds of training and scoring (two products for the first layer, three for the others, one when
    scoring), every input and every suggestion's record read once, every output written once.  Early stopping is
    counted up to the first epoch at which it can end a run."""
    n, d, K = case["rows"], case["features"], case["folds"]
    held = n / K
    fits = 1 if case["entry"] == "holdout" else K
    epochs = case["epochs"]
    fit_rows = n - held
    watched = 0.0
    if case["patience"]:
        epochs = min(epochs, case["patience"] + 2)
        watched = fit_rows * case["val_fraction"] * epochs
        fit_rows *= 1.0 - case["val_fraction"]
    c_out = max(case["classes"], 1)
    flops = 0.0
    for hidden, _ in _shapes(case):
        dims = [d] + hidden + [c_out]
        forward = sum(2.0 * a * b for a, b in zip(dims, dims[1:]))
        train = float(inputs.flops_per_sample(d, hidden, c_out))
        flops += fits * (train * fit_rows * epochs + forward * (held + watched))
    outputs = 3 + (2 * K if case["entry"] == "per_fold" else 0)
    return {"bytes": n * d * (2 if case["bf16"] else 4) + 8.0 * n + case["suggestions"] * (88.0 + 4.0 * outputs),
            "flops": flops}


def tolerance(case):
    """Scores are means over held rows of a model trained by hundreds of steps: what rounding does to the sums
    grows along the run.  "max" leaves room for single rows whose predicted class sits on the border (accuracy
    moves by one row) and, under early stopping, for a run that ends an epoch apart because two epochs' losses
    agree to rounding."""
    if case["bf16"]:
        return {"rel": 5e-3, "max": 0.05}
    if case["patience"]:
        return {"rel": 1e-3, "max": 0.05}
    return {"rel": 1e-4 if case["batch_hi"] == 0 else 3e-4, "max": 0.02}
