"""The autotuner times each candidate on the kernels that the candidate is about:
tiles, rows and column passes on the integer transforms, the schoolbook threshold
against the default ones."""
import pytest

pytestmark = pytest.mark.gpu

INTEGER = {"k_ntt_lds", "k_row", "k_crt"}
FP64 = {"k_flds", "k_frow", "k_ffused", "k_fcrt"}


def test_candidates_run_their_kernels(monkeypatch):
    import torch

    import paper_2601_11621_amd as cat
    from paper_2601_11621_amd import tune

    torch.cuda.set_device(0)
    seen = []
    real = tune._time_plan

    def spy(c, a_off, b_off, da, db, out, reps):
        plan = c.MulPlan(a_off, b_off, mode="batched")
        ran = set()
        for k in sorted(INTEGER | FP64 | {"k_school"}):
            c.timer_set(k)
            plan(da, db, out)
            plan.check()
            if c.timer_get()[1]:
                ran.add(k)
        c.timer_set(None)
        plan.close()
        seen.append(ran)
        return real(c, a_off, b_off, da, db, out, reps)

    monkeypatch.setattr(tune, "_time_plan", spy)
    try:
        res = tune.autotune(max_k=16, min_k=7, reps=1, total_log2=16, verbose=True)
        names = [(k, n) for k, ms in res["ms"].items() for n in ms]
        assert len(names) == len(seen)
        for (k, name), ran in zip(names, seen):
            print(k, name, sorted(ran), flush=True)
            if name == "school":
                assert ran == {"k_school"}, (k, ran)
            elif name == "fp64":
                assert ran and ran <= FP64, (k, ran)
            else:
                assert ran <= INTEGER, (k, name, ran)
                assert ("k_row" in ran) == name.startswith("rows"), (k, name, ran)
        assert all("fp64" in ms and ("school" in ms) == (k <= 8) for k, ms in res["ms"].items())
    finally:
        cat.timer_set(None)
        cat.set_integer_transforms(False)
        cat.set_tuning(None)
        cat.load_tuning()
