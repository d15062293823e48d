"""The benchmark's printed line: its figures at the head as measured, and short
enough for readers that keep the end of a run's output."""
import importlib.util
import json
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def load():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    return b


def document():
    """As the default run builds it, every figure at full length."""
    x = 123456.78901234567
    stages = {k: {"ms_per_window": x, "regions": 512}
              for k in ("rng", "proposal", "target", "step", "merge", "chol", "whiten", "psrf")}
    flat = {k: x for k in stages}
    moments = {f"{n}_{m}": dict.fromkeys(("estimate", "exact", "se", "z", "se_chains", "z_chains"), x)
               for n in ("logpi", "v_max", "v_min") for m in ("mean", "variance")}
    moments.update(worst_abs_z=x, worst_abs_z_chains=x, windows=196, samples_per_chain=50176, seconds=x)
    run = {"beta": 0.5, "alpha": 1.0, "delayed_acceptance": True, "seconds": x, "chain_steps_per_s": x,
           "ess": dict.fromkeys(("logpi", "v_max", "v_min"), x), "ess_per_s": x, "acceptance": x,
           "stage_ms_per_window": flat, "stage1_pass_rate": x, "stage2_accept_rate": x, "ess_per_s_incl_training": x,
           "surrogate": {"pairs": 50000, "adam_steps": 3000, "batch": 256, "final_loss": x, "train_seconds": x}}
    gain = {f"beta={b},alpha={a}": x for b, a in ((0.5, 1.0), (1.0, 1.0), (1.0, 1.2), (1.0, 1.5))}
    fam = {"ess_per_s": x, "ess_per_step": [x] * 3, "chain_steps_per_s": x, "beta": x}
    rates = {"chain_steps_per_s": x, "ess_per_s": x, "ms_per_window": x, "acceptance": x}
    text = "w" * 200
    return {"metric": "m" * 80, "value": x, "unit": "chain-steps/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": x, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
            "data": "synthetic", "config": {"workload": text, "d": 4096}, "ess_per_s": x, "steps_per_s": x,
            "acceptance": x, "stage_ms_per_window": stages,
            "roofline": {"kernel": text, "achieved": x, "frac": x, "work": text, "proposal": {"kernel": text, "frac": x}},
            "moments": moments, "moments_fixed_proposal": moments,
            "fp64": dict(rates, moments=moments, moments_fixed_proposal=moments, stage_ms_per_window=flat),
            "speedup_vs_fp64": {"chain_steps": x, "ess": x},
            "learned": {"workload": text, "runs": [run] * 8, "ess_per_s_gain_at_setting": gain,
                        "ess_per_exact_eval_gain_at_setting": gain},
            "batch": dict(rates, workload=text, ess={"note": text, "worst": moments}, persistent=dict(rates, note=text)),
            "families": {"workload": text, "targets": {t: dict.fromkeys(("diam", "am", "pcn", "rw"), fam)
                                                       for t in ("pi1", "pi2", "pi4", "pi4s", "pi5")}},
            "d1024": {"workload": text, "precisions": dict.fromkeys(("fp64", "fp32", "mixed"), rates)},
            "local_global": {"workload": text, "M": dict.fromkeys("14", dict(rates, stage_ms_per_window=flat))},
            "cpu_baseline": {"value": x, "unit": "chain-steps/s", "cores": 16, "kind": "oracle", "sample": text,
                             "host": {"cpu_model": text}, "note": text}}


def test_line_is_short_and_its_head_exact():
    doc = document()
    line = json.dumps(load().short(doc), separators=(",", ":"))
    got = json.loads(line)
    assert len(json.dumps(doc)) > 15000 and len(line) < 6500 and "\n" not in line
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config"):
        assert got[k] == doc[k]
    assert list(got)[:13] == list(doc)[:13]
    assert got["stage_ms_per_window"]["target"] == 123500.0 and got["fp64"]["stage_ms_per_window"]["rng"] == 123500.0
    assert got["speedup_vs_fp64"] == {"chain_steps": 123500.0, "ess": 123500.0}
    assert got["moments"] == {"worst_abs_z": 123500.0, "worst_abs_z_chains": 123500.0, "windows": 196}
    assert got["cpu_baseline"]["value"] == doc["cpu_baseline"]["value"]
