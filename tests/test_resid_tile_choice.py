"""The blocks of 64 columns on eight waves that residual projections of some hundred rows run in, where the library takes them and where it
does not, held against the measured times of every form that computes such a projection (profiles/resid_tile_times.txt).  Host code of the
built library; no GPU."""
import os

import test_tile_choice as large

FILE = os.path.join(large.ROOT, "profiles", "resid_tile_times.txt")


def test_what_runs_is_near_the_best_of_the_measured_forms():
    # Bounds: as for the large tiles.  Not in a large tile either where the choice falls to those.
    from paper_2605_26606_amd import binding
    lib = binding.library()
    regret, taken = [], 0
    for line in open(FILE):
        head, _, forms = line.partition("|")
        if len(head.split()) != 5 or "=" not in forms:
            continue
        launch, m, n, k, mode = head.split()
        m, n, k = int(m), int(n), int(k)
        times = {f.rsplit("=", 1)[0]: float(f.rsplit("=", 1)[1]) for f in forms.split()}
        tile = lib.pc_internal_resid_tile(m, n, k)
        taken += tile > 0
        form = [None, "m64x64", "m128x64"][tile] or large._chosen(lib, large.RESID, m, n, k, mode)
        late = times[form] / min(times.values())
        assert late <= (1.15 if k >= 1024 else 1.4), (launch, m, n, k, form, late)
        regret.append(late)
    assert len(regret) > 30 and 30 < taken < len(regret)
    assert sum(regret) / len(regret) <= 1.02
