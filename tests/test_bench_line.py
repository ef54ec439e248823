"""The benchmark's printed line (CPU only): short enough to survive whole, with the contract's keys."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

X = 1234.5678901234567


def _solution():
    leg = dict(precond_storage="fp64", status=0, converged=True, solve_ms=X, total_ms=X, newton=12, gmres=1234,
               jv_evals=1234, residual_evals=123, fnorm_inf=X, max_dzeta_vs_oracle=X, max_dphi_vs_oracle=X)
    P = dict(setup_ms=X, linear_start_ms=X, linear_start_prec="fp64", linear_start_rtol=X, band_halfwidth=10,
             bytes=10 ** 10, apply_ms=X, apply_GBps=X)
    row = dict(froude=0.6, precond_fp64=P, precond_fp32=P, workload="w" * 120, pairs_per_eval=10 ** 9,
               fp32c_vs_fp64=dict(max_dzeta_x=X, max_dphi_x=X))
    for name in ("fp64", "fp32c", "fp32c_p64", "fp32c_strict", "fp64_rtol1e-2"):
        row[name] = leg
        row[f"speedup_{name}"] = row[f"speedup_{name}_total"] = X
    return row


def test_line_holds_the_contract_and_stays_short():
    batch = dict(ms=X, pairs_per_s=X * 1e9)
    summary = {k: X for k in ("n", "both_converged", "fallbacks", "linear_newton_mean", "learned_newton_mean",
                              "linear_gmres_mean", "learned_gmres_mean", "linear_ms_mean", "learned_ms_mean",
                              "linear_f0_mean", "learned_f0_mean", "max_dx_between_solutions")}
    contract = dict(metric="pair-interactions/s + time-to-converged-solve, 181x61 grid: FP64 vs mixed/learned", value=X,
                    unit="pair-interactions/s", n_gpus=1, steps=20, warmup=5, ms_per_step=X, higher_is_better=True,
                    scaling="weak", vs_baseline=None, dtype="f64", data="synthetic",
                    config=dict(workload="w" * 110, pairs_per_eval=969928560))
    out = dict(contract,
               roofline=dict(bound="alu", achieved=X, peak=78.6, unit="TFLOP/s", frac=X, traffic=X,
                             kernel="k_s2_sums + k_allpairs64", kernel_ms=X, flop_per_pair=20.0),
               fp32c=dict(eval_ms=X, kernel_ms=X, pairs_per_s=X, roofline=dict(bound="alu", achieved=X, peak=157.3,
                                                                               unit="TFLOP/s", frac=X)),
               fp64_eval_ms_events=X, residual_evals_per_s=X,
               time_to_solution=[_solution() for _ in range(3)], time_to_solution_extended_domain=_solution(),
               time_to_solution_full_domain=_solution(),
               sweep=dict(grids=["100x34"] * 64, batched_residual_fp64=batch, batched_residual_fp32c=batch,
                          sweep=dict(precond_setup_s=X, linear_starts_s=X, batched_solve_s=X, converged=34,
                                     newton_total=341, gmres_total=23229, per_instance=[["sweep0-0", X, 3, 4, 385]] * 64)),
               exact_linear=dict(meshes=[dict(name=f"fig8-inline-281x281-F0.{i}", total_ms=X, contract_tflops=X,
                                              nodes=10 ** 6) for i in range(3)],
                                 newton_from_exact_start_181x61=[dict(a=[X] * 40)] * 2),
               learned_start_121x41=dict(mesh="121x41", summary=summary),
               cpu_baseline=dict(value=X, unit="pair-interactions/s", cores=16, kind="oracle", sample="s" * 130))
    line = json.dumps(bench.headline(out))
    print(len(line))
    assert len(line) <= 5000
    back = json.loads(line)
    for k, v in contract.items():
        assert back[k] == v, k
    assert json.dumps(bench.headline(contract)) == json.dumps(contract)  # no legs: the timed steps alone
