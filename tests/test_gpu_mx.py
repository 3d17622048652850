"""GPU parity of the MXFP4 expert path (through the C ABI) against the oracle.

Weights are MXFP4, activations and h MXFP8 (the oracle mirrors both
quantisations); outputs are held to the e4m3 relative-RMS bound.

* reduced DeepSeek-V4-Flash-shaped workload over every row, both M tiles
* full-size workload on sampled tokens, hottest and coldest experts included
* 128-row and 256-row M tiles give the same bits; a fetched expert equals a
  resident one; a zero-gate expert gives exact zeros
* the persistent 256-row tiles over more tiles than workgroups, with an odd
  number of GEMM2 K steps, on every row and bitwise equal to 128-row tiles;
  with fetched experts (their own persistent launches) bitwise equal to the
  all-resident layer
"""
import numpy as np
import pytest
import torch

from paper_2609_33252_amd import cep, harness, workload as W

from . import _util as U

pytestmark = pytest.mark.gpu

NAME = "mxfp4_dsv4flash_d4096"
# the oracle finishes this in seconds: 8 experts of 2048 x 1024, ~1.5k pairs
SMALL = dict(d=2048, I=1024, E=8, Eg=64, R=4, T=512, cpr=4)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cep.lib()
    torch.cuda.set_device(0)


def _out(run):
    torch.cuda.synchronize()
    cep.cep_get_status(run.ctx)
    return run.out.cpu().numpy()


def test_mxfp4_reduced_all_rows():
    wl = W.generate(NAME, 0, **SMALL)
    run = harness.Runner(wl, n_streams=2, record_routing=True)
    run.run(policy=cep.CEP_THRESHOLD, theta=max(1, wl.n_pairs // 3), n_streams=2)
    got = _out(run)
    aligns = {cep.cep_get_batch_routing(run.ctx, b, wl.cfg["E"], wl.cfg["k"])["align"]
              for b in range(cep.cep_get_batch_count(run.ctx))}
    run.close()
    mx, rel = U.check(wl, got)
    assert not got[~wl.delivered].any()
    print(f"mxfp4 reduced: pairs={wl.n_pairs} aligns={sorted(aligns)} max_abs={mx:.3e} "
          f"rel_rms={rel:.3e}")


def test_mxfp4_large_and_small_m_tiles_agree_bitwise():
    # wait-all: >= 256 rows per expert (256-row tile); per chunk: 64-row tiles
    wl = W.generate(NAME, 1, d=1024, I=512, E=4, Eg=32, R=4, T=2048, cpr=8)
    assert wl.n_pairs >= 256 * wl.cfg["E"]
    run = harness.Runner(wl, n_streams=2, record_routing=True)
    run.run(policy=cep.CEP_WAIT_ALL)
    a = _out(run)
    assert cep.cep_get_batch_routing(run.ctx, 0, wl.cfg["E"], wl.cfg["k"])["align"] == 256
    run.out.zero_()
    run.run(policy=cep.CEP_PER_CHUNK, n_streams=2)
    b = _out(run)
    assert cep.cep_get_batch_routing(run.ctx, 0, wl.cfg["E"], wl.cfg["k"])["align"] == 128
    run.close()
    assert np.array_equal(a, b)
    U.check(wl, a)


def test_mxfp4_full_size_sampled_tokens():
    wl = W.generate(NAME, 0)
    run = harness.Runner(wl, n_streams=1)
    run.run(policy=cep.CEP_WAIT_ALL)
    got = _out(run)
    run.close()
    rng = np.random.default_rng(2)
    deliv = np.argwhere(wl.delivered)
    pick = deliv[rng.choice(len(deliv), size=16, replace=False)]
    cnt = np.bincount(wl.topk_local[wl.topk_local >= 0], minlength=wl.cfg["E"])
    for e in (int(cnt.argmax()), int(np.argmin(np.where(cnt > 0, cnt, 1 << 30)))):
        rt = np.argwhere((wl.topk_local == e).any(axis=2))
        pick = np.vstack([pick, rt[-2:]])
    mx, rel = U.check(wl, got[pick[:, 0], pick[:, 1]], tokens=pick)
    assert not got[~wl.delivered].any()
    print(f"mxfp4 full: pairs={wl.n_pairs} sampled={len(pick)} max_abs={mx:.3e} rel={rel:.3e}")


def test_mxfp4_fetched_experts_equal_resident_bitwise():
    wl = W.generate(NAME, 3, **dict(SMALL, fetch_frac=0.25))
    assert wl.fetched
    a = harness.Runner(wl, n_streams=2, use_fetch=True)
    a.run(policy=cep.CEP_THRESHOLD, theta=500, n_streams=2)
    ga = _out(a)
    assert all(b["fetched"] for b in a.stats()["batches"])
    a.close()
    b = harness.Runner(wl, n_streams=1, use_fetch=False)
    b.run(policy=cep.CEP_WAIT_ALL)
    gb = _out(b)
    b.close()
    assert np.array_equal(ga, gb)


def test_mxfp4_zero_gate_codes_give_exact_zero():
    # all gate codes of expert 0 are +0: gate = 0, silu(0) * up = 0, h = 0,
    # so every row routed only to expert 0 comes out exactly 0
    wl = W.generate(NAME, 4, d=1024, I=512, E=4, Eg=8, R=2, T=256, cpr=2)
    wg = wl.w_gate.clone()
    wg[0] = 0
    wl.w_gate = wg
    only0 = np.where(wl.topk_local == 0, 0, -1).astype(np.int32)
    wl.topk_local = only0
    run = harness.Runner(wl, n_streams=1)
    run.run(policy=cep.CEP_WAIT_ALL)
    got = _out(run)
    run.close()
    assert wl.n_pairs > 0
    assert not got.any()


def test_mxfp4_persistent_tiles_odd_k_steps_all_rows():
    # The persistent 8-wave MXFP4 tiles over more tiles than workgroups (each
    # workgroup runs several, loading the next one's first stage and GEMM2
    # coefficients during the epilogue) with an odd number of GEMM2 K steps
    # (I = 640: five), so that a tile's last step uses ring buffer 0, the
    # buffer the next tile's first stage fills: every row against the oracle,
    # and bitwise equal to per-chunk batches on the 64-row tiles.
    wl = W.generate(NAME, 12, d=1024, I=640, E=4, Eg=16, R=4, T=4096, cpr=64)
    E, k = wl.cfg["E"], wl.cfg["k"]
    run = harness.Runner(wl, n_streams=1, record_routing=True, use_fetch=False)
    run.run(policy=cep.CEP_WAIT_ALL)
    a = _out(run)
    m = cep.cep_get_batch_routing(run.ctx, 0, E, k)
    assert m["align"] == 256
    m_tiles = int(sum((c + 255) // 256 for c in m["cnt"]))
    assert m_tiles * (wl.cfg["d"] // 256) > 256, m["cnt"]  # GEMM2 tiles > workgroups
    mx, rel = U.check(wl, a)
    run.out.zero_()
    run.run(policy=cep.CEP_PER_CHUNK)
    b = _out(run)
    aligns = {cep.cep_get_batch_routing(run.ctx, i, E, k)["align"]
              for i in range(cep.cep_get_batch_count(run.ctx))}
    run.close()
    assert aligns == {128}
    assert np.array_equal(a, b)
    print(f"mxfp4 persistent tiles, odd K steps: pairs={wl.n_pairs} max_abs={mx:.3e} rel={rel:.3e}")


def test_mxfp4_persistent_tiles_fetched_equal_resident_bitwise():
    # 256-row batches with fetched experts: the resident and the fetched
    # experts' tiles run as two persistent launches per GEMM (the fetched
    # ones behind the copy); bitwise equal to every expert resident.
    wl = W.generate(NAME, 13, d=1024, I=640, E=8, Eg=32, R=4, T=4096, cpr=64, fetch_frac=0.25)
    assert wl.fetched
    E, k = wl.cfg["E"], wl.cfg["k"]
    a = harness.Runner(wl, n_streams=1, record_routing=True, use_fetch=True)
    a.run(policy=cep.CEP_WAIT_ALL)
    ga = _out(a)
    assert cep.cep_get_batch_routing(a.ctx, 0, E, k)["align"] == 256
    assert all(b["fetched"] for b in a.stats()["batches"])
    a.close()
    b = harness.Runner(wl, n_streams=1, use_fetch=False)
    b.run(policy=cep.CEP_WAIT_ALL)
    gb = _out(b)
    b.close()
    assert np.array_equal(ga, gb)
    mx, rel = U.check(wl, gb)
    print(f"mxfp4 persistent tiles with fetched experts: pairs={wl.n_pairs} rel={rel:.3e}")
