"""sv_run_stats.bytes of a batch counts 16 * 2^n per pass, whatever a tuning
file says about the LDS limit that files of earlier versions carry; such a file
still loads, and a limit out of range is still refused."""
import json

import pytest

import circuits as C

pytestmark = pytest.mark.gpu


def test_bytes_do_not_depend_on_the_file(tmp_path):
    from paper_2602_09604_amd import sv
    ns, circs = C.batched_ansatz(8, seed=5, n_min=9, n_max=14)
    states = [sv.State(n) for n in ns]
    try:
        want = sum((16 << n) * len(sv.sv_fuse(c, n, sv.make_opts(max_k=4))[0]) for n, c in zip(ns, circs))
        for limit in (None, 1, 12, 14):
            if limit is not None:
                p = tmp_path / "t.json"
                p.write_text(json.dumps({"format": "libsv-tune-1", "batch_lds_max_n": limit, "entries": []}))
                sv.sv_tune_load(str(p))
            assert sv.sv_batch_run([s.h for s in states], circs, sv.make_opts(max_k=4))["bytes"] == want, limit
        p.write_text(json.dumps({"format": "libsv-tune-1", "batch_lds_max_n": 15, "entries": []}))
        with pytest.raises(sv.SvError) as e:
            sv.sv_tune_load(str(p))
        assert e.value.code == sv.SV_EINVAL
    finally:
        for s in states:
            s.free()
