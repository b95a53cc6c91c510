"""What bench.py times: the steps as a program runs them, and the stage times in a pass of their own."""
import json
import sys

import pytest

pytestmark = pytest.mark.gpu


def test_timed_steps_run_without_stage_timing(monkeypatch, capsys):
    import bench
    from paper_2605_17889_amd import binding as B
    armed, steps = [False], []

    def watch(name, before):
        call = getattr(B, name)

        def wrapped(*args, **kw):
            before()
            return call(*args, **kw)
        monkeypatch.setattr(B, name, wrapped)

    watch("moe_profile_begin", lambda: armed.__setitem__(0, True))
    watch("moe_profile_end_per_call", lambda: armed.__setitem__(0, False))
    watch("moe_layer_forward", lambda: steps.append(armed[0]))
    monkeypatch.setattr(sys, "argv", ["bench.py", "--workload", "tiny", "--steps", "5", "--warmup", "2",
                                      "--no-cpu-baseline"])
    print("bench.py on the smallest layer, in this process", flush=True)
    bench.main()
    out = json.loads(capsys.readouterr().out.strip().splitlines()[-1])
    assert steps == [False] * (2 + 5) + [True] * 5
    assert out["steps"] == 5 and out["ms_per_step"] > 0
    assert all(out["stages"][s]["ms_per_step"] > 0 for s in ("route", "permute", "gateup", "down", "combine"))
