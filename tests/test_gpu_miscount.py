"""Chunks whose ids hold more pairs than their n_pairs says: the library reports
them (cep_get_status), stays inside its buffers, and the calls that follow are
right.  (Which loads a miscounted batch may issue is checked on the CPU,
tests/test_host_native.py.)"""
import numpy as np
import pytest
import torch

from paper_2609_33252_amd import cep, harness, workload as W

from . import _util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cep.lib()


def _workload(name, d, I, cnt, T):
    """One chunk of T rows whose slot 0 gives the experts the counts cnt."""
    E = len(cnt)
    wl = W.generate(name, 3, d=d, I=I, E=E, Eg=E, k=2, R=1, T=T, cpr=1, fetch_frac=0.0)
    ids = np.full((T, 2), -1, np.int32)
    own = np.repeat(np.arange(E, dtype=np.int32), cnt)
    ids[:len(own), 0] = own[np.random.default_rng(5).permutation(len(own))]
    wl.topk_local = ids.reshape(1, T, 2)
    return wl


def _part(ch, n):
    """The first n rows of a chunk, rightly counted."""
    p = harness.DeviceChunk()
    p.replica, p.n_rows, p.arrival_ms = ch.replica, n, 0.0
    p.token_idx, p.x, p.ids, p.w = ch.token_idx[:n], ch.x[:n], ch.ids[:n], ch.w[:n]
    p.n_pairs = int((p.ids >= 0).sum().item())
    return p


def test_tile_in_the_last_scale_group():
    # e4m3, 160-row tiles: 3552 pairs declared as 2000 fill the context's 4352
    # grouped rows to the last; the tile at row 4224 lies in the last 128-row
    # group of the row scales
    wl = _workload("fp8_fetch_d6144", 256, 2048, [160] * 5 + [400] * 2 + [1952], 4096)
    run = harness.Runner(wl, n_streams=1, use_fetch=False, max_pairs=2000)
    run.chunks[0].n_pairs = 2000
    run.run(policy=cep.CEP_WAIT_ALL)
    with pytest.raises(cep.CepError) as e:
        cep.cep_get_status(run.ctx)
    assert "n_pairs mismatch" in str(e.value) and "capacity" not in str(e.value)
    run.chunks.append(_part(run.chunks[0], 1200))
    run.out.zero_()
    run.run_subset([1])
    torch.cuda.synchronize()
    cep.cep_get_status(run.ctx)
    got = run.out.cpu().numpy()
    run.close()
    tok = np.stack([np.zeros(1200, np.int64), np.arange(1200)], axis=1)
    U.check(wl, got[0, :1200], tokens=tok)


@pytest.mark.parametrize("T", [1024, 4096], ids=["one-block routing", "two-kernel routing"])
@pytest.mark.parametrize("call", ["layer", "noalloc"])
@pytest.mark.parametrize("name", ["sync_d4096", "tiny", "fp8_fetch_d6144",
                                  "mxfp4_dsv4flash_d4096"])
def test_batch_beyond_its_buffers_runs_no_tile(name, call, T):
    # 1007 pairs declared as 100: more tiles, and without a context's slack more
    # grouped rows, than the buffers hold.  Every token has one local pair, whose
    # output row GEMM2 itself would write: rows stay as they were, or are zero
    # where the pair has no grouped row
    wl = _workload(name, 256, 128, [1] * 7 + [1000], T)
    run = harness.Runner(wl, n_streams=1, use_fetch=False, max_pairs=100)
    ch = run.chunks[0]

    def go(c):
        run.out.fill_(5.0)
        if call == "noalloc":
            cep.cep_ffn_noalloc(run.ctx, c.replica, c.n_rows, c.n_pairs, c.token_idx, c.x, c.ids,
                                c.w, run.out, torch.cuda.current_stream())
        else:
            run.run_subset([run.chunks.index(c)])
        torch.cuda.synchronize()

    ch.n_pairs = 100
    go(ch)
    with pytest.raises(cep.CepError) as e:
        cep.cep_get_status(run.ctx)
    assert "n_pairs mismatch" in str(e.value) and "capacity" in str(e.value)
    out = run.out[0, :1007].cpu().numpy()
    assert np.all((out == 5.0).all(axis=1) | (out == 0.0).all(axis=1))
    run.chunks.append(_part(ch, 90))
    go(run.chunks[1])
    cep.cep_get_status(run.ctx)
    got = run.out.cpu().numpy()
    run.close()
    tok = np.stack([np.zeros(90, np.int64), np.arange(90)], axis=1)
    U.check(wl, got[0, :90], tokens=tok)
    assert np.all(got[0, 90:] == 5.0)
