"""The benchmark's passes: every index map once, the headline's with the fastest."""
import bench


def test_only_the_fastest_map_takes_the_timed_passes():
    rate = {"clt": 3.0, "cr": 4.0, "full": 1.0, "lin": 2.0}
    calls = []

    def measure(mode, warmup, steps, first):
        calls.append((mode, warmup, steps))
        return {"states_bonds_per_s": rate[mode], "passes": steps, "autotune_ms": {"8": 1.0} if first else {},
                "hv_width_sweep": {"1": mode} if first else {}}

    best, results = bench.run_passes(list(rate), 5, 20, measure)
    assert best == "cr" and set(results) == set(rate)
    # 20 timed passes after 5 untimed ones, and one of each map: 4 + 25, not 4 x 25
    assert sum(w + k for _, w, k in calls) == len(rate) + 25
    assert calls[-1] == ("cr", 5, 20)
    assert results["cr"]["passes"] == 20 and results["cr"]["hv_width_sweep"] == {"1": "cr"}
    assert results["cr"]["autotune_ms"] == {"8": 1.0}
    assert all(results[m]["passes"] == 1 for m in rate if m != "cr")
