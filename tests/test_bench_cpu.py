"""The bench line's first-stage roofline follows the form that the plan runs."""

import importlib.util
import os

import numpy as np

import synth
import paper_2401_13834_amd as tx

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
spec = importlib.util.spec_from_file_location("tx_bench", os.path.join(ROOT, "bench.py"))
bench = importlib.util.module_from_spec(spec)
spec.loader.exec_module(bench)


def counted(plan):
    """The products one by one, over their full number."""
    i, t = plan.info, plan.tables()
    g, nsub, m = i["ngroups"], i["nsub"], i["chans_per_sub"]
    n = 0
    for s in range(nsub):
        for j0 in range(0, g, 16):
            for c0 in range(0, m, 4):
                for j4 in range(j0, j0 + 16, 4):
                    most = 0
                    for c in range(c0, min(c0 + 4, m)):
                        d = [int(t["coarse_chan"][min(j, g - 1), s * m + c] - t["coarse_sub"][min(j, g - 1), s])
                             for j in range(j0, j0 + 16)]
                        mine = d[j4 - j0:j4 - j0 + 4]
                        start = min(d) // 16 * 16
                        most = max(most, max(mine) - start - (min(mine) - start) // 4 * 4)
                    n += 1 + (most + 7) // 16
    return n / (g / 4 * nsub * m / 4)


def test_products():
    for nchan, nsub, ndm, step, g in [(96, 8, 40, 3.0, 1), (84, 12, 17, 10.0, 1), (64, 4, 200, 0.7, 4)]:
        plan = tx.tx_plan(synth.band_centres(1712.0, 856.0, nchan), 256e-6, np.arange(ndm) * step, nsub,
                          dms_per_group=g, host_only=True)
        assert abs(bench.mx_windows(plan) - counted(plan)) < 1e-9


def test_forms():
    f = synth.band_centres(1712.0, 856.0, 1024)
    for step, bound in ((0.1, "mfma"), (60.0, "alu")):
        plan = tx.tx_plan(f, 153.12e-6, np.arange(128) * step, 16, dms_per_group=1, host_only=True)
        r = bench.stage1_roofline(tx, plan, 16384, 40.0)
        assert r["bound"] == bound and r["achieved"] == 40.0 and 0.0 < r["frac"] < 1.0
        assert r["loop_ceiling_frac"] == round(40.0 / r["loop_ceiling_Tadd_s"], 4) or abs(
            r["loop_ceiling_frac"] - 40.0 / r["loop_ceiling_Tadd_s"]) < 1e-3
