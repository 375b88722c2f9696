"""Tuned blocks per launch of short blocks: the tuner tries what an untuned plan or
search launches, so asking it to measure is not slower than not asking; choices
stored without those candidates are measured again."""
import numpy as np
import pytest

import synth
from gpu_helpers import BW, F0

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["fp32", "half"])
def test_tuned_short_blocks(form, tmp_path, monkeypatch):
    import torch
    import paper_1503_01405_amd as P
    cache = tmp_path / "tune.txt"
    prop = torch.cuda.get_device_properties(0)
    tag = f"{prop.gcnArchName.split(':')[0]}-{prop.multi_processor_count}cu"
    cache.write_text("".join(
        f"pond-tune-4 {tag} {path} nfft=4096 form={P.FORMS[form]} kind=0 hist=lds batch=16 ms_per_block=0.001000 "
        "default_batch=16 default_ms_per_block=0.001000\n" for path in ("dedisperse", "search2")))
    monkeypatch.setenv("POND_AUTOTUNE_CACHE", str(cache))
    x = torch.from_numpy(synth.white_stream_int8(101, 3_000_001)).cuda()
    outs = []
    for batch in (P.POND_BATCH_AUTOTUNE, 0, P.POND_BATCH_AUTOTUNE):
        plan = P.Plan(F0, BW, 0.03, 1 << 12, 64, 0.0053, precision=form, max_batch=batch, subint_nsamp=0, decim=16)
        if batch:
            r = plan.autotune()
            print(form, r, flush=True)
            # 32 blocks of 2^12 leave three CUs in four idle: several times slower
            assert r["batch"] > 32 and r["from_cache"] == (len(outs) == 2)
            assert r["ms_per_block"] < 0.5 * r["default_ms_per_block"]
        outs.append([plan.process(x)[1].cpu().numpy(), plan.flush().cpu().numpy()])
        plan.close()
    for got in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(got, outs[0]))
    profs = []
    for batch in (P.POND_BATCH_AUTOTUNE, None):
        h = P.pond_search_create(F0, BW, [0.0, 0.01, 0.02], 64, 0.0053, 1 << 12, 1 << 12, P.FORMS[form], max_batch=batch)
        if batch:
            r = P.pond_search_autotune(h, 1 << 12)
            print(form, r, flush=True)
            assert r["batch"] > 32 and not r["from_cache"]
        prof = torch.empty(3, 64, device="cuda")
        assert P.pond_search_run(h, x, 3_000_001, prof) == P.POND_OK
        profs.append(prof.cpu().numpy())
        P.pond_search_destroy(h)
    assert np.array_equal(profs[0], profs[1])
