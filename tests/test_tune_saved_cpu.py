"""What a tuning run saves: its selection where the step is faster with it,
the library's own choices otherwise."""
from paper_2007_00072_amd import lib, tune


def result(planned):
    entry = lib.ContractChoice(4096, 3072, 1024, 1, lib.DM_F16, 1, 1, 25, 1)
    own = [lib.ContractChoice(4096, 3072, 1024, 1, lib.DM_F16, 1, 1, 27, 1)] * 2
    return {"workload": "bert_large_f16", "attn_path": 3, "qkv_fusion": 1, "entries": tune.as_dicts([entry]),
            "own_entries": tune.as_dicts(own), "builtin_ms": 0.6, "planned_ms": planned,
            "layout": {"ln_bwd_form": 2, "dO_transposed": 1, "dH_transposed": 0, "ln_lanes": 32}}


def test_faster_selection_is_saved():
    res = result(0.55)
    plan = tune.to_save(res)
    assert plan == {k: v for k, v in res.items() if k != "own_entries"}


def test_slower_selection_is_not_saved():
    plan = tune.to_save(result(0.6))
    assert [e["tile_cfg"] for e in plan["entries"]] == [27]
    assert plan["attn_path"] == 0 and plan["qkv_fusion"] == 0 and set(plan["layout"].values()) == {-1}
    assert "own_entries" not in plan
    lib.Plan([lib.ContractChoice(*[e[f] for f in ("M", "N", "K", "batch", "dtype", "a_kcontig", "b_kcontig", "tile_cfg",
                                                  "splits")]) for e in plan["entries"]], plan["attn_path"], plan["layout"])
