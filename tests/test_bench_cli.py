"""Host-side checks of bench.py's workload grammar (no GPU): each spec builds the workload it
names, with its block shape, density, token count and dtype, and specs a workload cannot honour
are refused instead of silently measuring something else."""
import json

import pytest

import bench


def _shape(wl):
    p = wl.projections[0]
    return p.R, p.C, p.W.shape


def test_fused_qkv_spec():
    wl = bench.build_workload("fused_qkv:16x16:0.2:bf16")
    assert wl.bf16 and wl.tokens == 4096
    assert _shape(wl) == (16, 16, (2304, 768))
    assert wl.projections[0].density == pytest.approx(0.2)


def test_ffn_spec_density_tokens_dtype():
    wl = bench.build_workload("ffn:32x1:0.05:256")
    assert not wl.bf16 and wl.tokens == 256
    assert [p.W.shape for p in wl.projections] == [(3072, 768), (768, 3072)]
    assert all(p.density == pytest.approx(0.05) for p in wl.projections)
    assert bench.build_workload("ffn:32x32:bf16").bf16


def test_reblock_spec():
    wl = bench.build_workload("sweep:64x64@32x32")
    assert wl.notes["reblock"] == (32, 32)
    assert _shape(wl)[:2] == (64, 64)


@pytest.mark.parametrize("spec", ["sweep:32x1:bf16", "bert_large:32x32:bf16", "nonsense:32x1"])
def test_refused_specs(spec):
    with pytest.raises(SystemExit):
        bench.build_workload(spec)


def test_result_line_stays_short():
    """The rows' part of the result line (31 product rows, two of the iterative projection) is a few
    KB: a reader of the last 8 KB of the output still gets the whole line."""
    def product(spec):
        return {"workload": "w" * 40, "spec": spec, "block": "32x1", "dtype": "f32",
                "tokens": 4096, "plans": True, "plan_arithmetic": "bf16x3 split",
                "products_per_launch": 1, "launches": 64, "protocol": "p" * 60,
                "launch_us": {k: 15.598000027239323 for k in ("median", "p10", "p90", "mean")},
                "loop_us_per_launch": 18.638359382748604, "effective_tflops": 45.75759343950161,
                "effective_tbs": 3.2010218200905394,
                "roof": {"bound": "mfma", "frac": 0.4001277275113174,
                         "arithmetic_intensity": 14.294683389008384},
                "frac_of_hbm": 0.4001277275113174, "frac_of_matrix_peak": 0.2908937917323688,
                "dense_us": {k: 134.00299847126007 for k in ("median", "p10", "p90")},
                "sparse_over_dense": 0.11640038062718919}
    iht = {"workload": "iht_bert_base_768_32x1_d10", "block": "32x1", "iterations": 20, "k": 1843,
           "eta": 0.00011985416935728542, "hessian": "X^T X of 4096 tokens",
           "us_per_iteration": 58.39089825749397, "setup_us": 126.50500237941742,
           "loss_one_shot": 412845.6202954926, "loss_after": 405065.82393485185,
           "cpu_oracle_ms_per_iteration": 3.5173723333343787}
    full = {"fused_qkv": [product("fused_qkv:32x1:0.05:bf16") for _ in range(31)],
            "iht_bert_base": [iht, iht]}
    short = bench.short_rows(full)
    assert len(json.dumps(short)) < 4500
    r = short["fused_qkv"][0]
    assert r["row"] == "fused_qkv:32x1:0.05:bf16 split" and r["us"] == 15.6
    assert short["iht_bert_base"][1]["loss_after"] == iht["loss_after"]
