"""Few-row tiles of the GEMMs at their edges: experts whose row
counts sit at the edges of the 8-row load segments, the 16-row fragments and
the 64-, 128- and 160-row tiles, every row against the oracle (the bounds of
_util.check).  The K loops have one, two, three, six and 22 steps.  Each case
states which tiles it runs (tests/_native.py evaluates the library's own rule),
so that a moved line between them cannot empty it."""
import numpy as np
import pytest
import torch

from paper_2609_33252_amd import cep, harness, workload as W

from . import _native as N
from . import _util as U

pytestmark = pytest.mark.gpu

# rows per expert: 64-row tiles (fewer than 64 pairs per expert on average, or
# few work items), and larger counts
COUNTS = {"rows64": [1, 8, 9, 16, 17, 0, 64, 65, 128, 129, 63, 7],
          "rows128": [127, 128, 129, 1, 112, 113, 0, 256, 257, 64, 15, 240],
          # with I 2816 the batch has enough work items for the larger tiles
          # (128 rows for bf16 and MXFP4, 160 for e4m3: tiles that start at row 32, 64 and 96 of a
          # 128-row scale group)
          "rows160": [159, 160, 161, 1, 320, 321, 0, 480, 15, 240, 176, 145]}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cep.lib()


@pytest.mark.parametrize("tiles", list(COUNTS))
@pytest.mark.parametrize("shape", [(768, 384), (256, 128)], ids=["d768", "d256"])
@pytest.mark.parametrize("name", ["fp8_fetch_d6144", "mxfp4_dsv4flash_d4096", "sync_d4096", "tiny"])
def test_row_counts_at_tile_edges(name, shape, tiles):
    cnt = COUNTS[tiles]
    E, (d, I) = len(cnt), shape
    if tiles == "rows160":
        I = 2816
    print(f"case {name} d={d} I={I} {tiles}", flush=True)
    # every expert local, so every token is delivered; then one local slot per
    # token up to the counts, and a second one (of the next expert) for some
    T = 4096
    wl = W.generate(name, 31, d=d, I=I, E=E, Eg=E, k=2, R=1, T=T, cpr=1, fetch_frac=0.0)
    ids = np.full((T, 2), -1, np.int32)
    own = np.repeat(np.arange(E, dtype=np.int32), cnt)
    order = np.random.default_rng(5).permutation(len(own))
    half = len(own) // 2
    ids[:len(own) - half, 0] = own[order[:len(own) - half]]
    rest = own[order[len(own) - half:]]
    both = rest != ids[:half, 0]  # a token's slots name distinct experts
    ids[:half, 1][both] = rest[both]
    ids[T // 2:T // 2 + int((~both).sum()), 0] = rest[~both]
    wl.topk_local = ids.reshape(1, T, 2)
    assert wl.n_pairs == sum(cnt)
    bf16 = name in ("sync_d4096", "tiny")
    few, more = ("64 by rows", "128") if bf16 else ("64", "160" if "fp8" in name else "128")
    assert N.tiles(wl, wl.n_pairs) == (more if tiles == "rows160" else few)
    run = harness.Runner(wl, n_streams=1, record_routing=True, use_fetch=False)
    run.run(policy=cep.CEP_WAIT_ALL)
    torch.cuda.synchronize()
    cep.cep_get_status(run.ctx)
    m = cep.cep_get_batch_routing(run.ctx, 0, E, 2)
    got = run.out.cpu().numpy()
    run.close()
    assert m["align"] == (64 if bf16 else 128) and list(m["cnt"]) == cnt
    U.check(wl, got)


# Shapes on both sides of the lines between the tile choices of a batch
# (batch_plan): few work items and many, for the pairs per expert at which the
# choice then differs, some with fetched experts (tile lists of their own).
# (preset, overrides, tokens per replica, tiles of the wait-all batch, of a
# quarter of it)
PLANS = [
    ("sync_d4096", dict(d=256, I=128, E=8, Eg=16, k=4), 256, "64 by rows", "64 by rows"),
    ("sync_d4096", dict(d=256, I=128, E=8, Eg=16, k=4), 800, "64 by rows", "64 by rows"),
    ("sync_d4096", dict(d=512, I=2048, E=16, Eg=32, k=2), 1200, "128", "64 by rows"),
    ("sync_d4096", dict(d=512, I=2048, E=16, Eg=32, k=2, fetch_frac=0.25), 1200, "128",
     "64 by rows"),
    ("sync_d4096", dict(d=256, I=2560, E=8, Eg=16, k=4), 640, "256", "128"),
    # (a last-bit difference of an h element can move its e4m3 code, by up to
    # 1/8 of the element: 3 sigma / 8 of a row of norm sigma sqrt(I), 3.3e-2 of
    # it at I = 128 beside the per-row bound of 4e-2, 1.7e-2 at I = 512)
    ("fp8_fetch_d6144", dict(d=256, I=512, E=8, Eg=16, k=4), 800, "64", "64"),
    ("fp8_fetch_d6144", dict(d=256, I=2560, E=8, Eg=16, k=4), 640, "256", "160"),
    ("fp8_fetch_d6144", dict(d=256, I=2560, E=8, Eg=16, k=4, fetch_frac=0.25), 640, "256", "160"),
    # 256-row tiles either side of the three rounds of work items up to which GEMM1
    # skips empty row fragments (500 and 600 rows per expert, 20 column tiles)
    ("fp8_fetch_d6144", dict(d=256, I=2560, E=16, Eg=32, k=4), 2000, "256", "160"),
    ("fp8_fetch_d6144", dict(d=256, I=2560, E=16, Eg=32, k=4), 2400, "256", "160"),
    ("mxfp4_dsv4flash_d4096", dict(d=256, I=512, E=8, Eg=16, k=4), 400, "64", "64"),
    ("mxfp4_dsv4flash_d4096", dict(d=256, I=2560, E=12, Eg=24, k=4), 300, "128", "64"),
    ("mxfp4_dsv4flash_d4096", dict(d=256, I=2560, E=12, Eg=24, k=4, fetch_frac=0.25), 300, "128",
     "64"),
    ("mxfp4_dsv4flash_d4096", dict(d=256, I=2560, E=8, Eg=16, k=4), 640, "256", "64"),
]


@pytest.mark.parametrize("i", range(len(PLANS)))
def test_tile_choice_lines(i):
    name, over, T, whole, part = PLANS[i]
    print(f"case {name} {over} T={T}", flush=True)
    wl = W.generate(name, 40 + i, **dict(dict(R=2, T=T, cpr=2, zipf=None, fetch_frac=0.0), **over))
    assert N.tiles(wl, wl.n_pairs) == whole
    assert {N.tiles(wl, wl.chunk_pairs(c)) for c in wl.chunks} == {part}
    run = harness.Runner(wl, n_streams=2)
    run.run(policy=cep.CEP_WAIT_ALL)
    torch.cuda.synchronize()
    cep.cep_get_status(run.ctx)
    a = run.out.cpu().numpy()
    run.out.zero_()
    run.run(policy=cep.CEP_PER_CHUNK, n_streams=2)  # smaller tiles, the same bits
    torch.cuda.synchronize()
    cep.cep_get_status(run.ctx)
    b = run.out.cpu().numpy()
    run.close()
    U.check(wl, a)
    assert np.array_equal(a, b)
