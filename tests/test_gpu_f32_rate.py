"""The fp32 products over many rows run at the rate that the card's vector units allow for a kernel of this kind: a tile
that is right for a few hundred rows can cost a third of it."""
import numpy as np
import pytest
import torch

from paper_2601_15013_amd import harness, synth

pytestmark = pytest.mark.gpu


def test_many_rows_keep_their_rate():
    # 65000 rows of the tiny fp32 model: 204.5 GFLOP of products.  On an MI355X the forward reaches 52 TFLOP/s of them with
    # 64x64 tiles of short k-tiles, 41 with the plain 64x64 kernel and 33 with k-tiles of 64; the bar is between.
    cfg = synth.TINY
    n, length = 65000, 8
    rng = np.random.default_rng(2)
    tok = torch.from_numpy(rng.integers(0, cfg.vocab, size=n, dtype=np.int32)).cuda()
    cu = torch.arange(0, n + 1, length, dtype=torch.int32, device="cuda")
    model = harness.upload_model(synth.SynthWeights(cfg, 3))
    try:
        run = harness.Runner(model, n, cu.numel() - 1)
        out = run.forward_nodedup(tok, cu, length)
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            run.forward_nodedup(tok, cu, length, out=out)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e-3)
        assert run.status() == 0
    finally:
        model.close()
    per_row = cfg.n_layers * (cfg.d * (cfg.dq + 2 * cfg.dkv) + cfg.dq * cfg.d + 3 * cfg.d * cfg.d_int)
    rate = 2.0 * n * per_row / float(np.median(times))
    assert rate > 38e12, f"{rate / 1e12:.1f} TFLOP/s"
