"""The automatic choice of a product's launch, on the CPU: the rule is host
arithmetic on sizes, strides and the number of compute units, so its routes can
be checked without a device (the bits of every route are the GPU tests')."""
import math
import os
import re

import pytest

from perf import gemm_choice

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2502_19405_amd", "librepops.so")
TIMINGS = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles",
                       "gemm_choice_timings.csv")


@pytest.fixture(scope="module")
def rp():
    if not os.path.exists(LIB):
        pytest.fail("librepops.so is not built (run python -m paper_2502_19405_amd.build)")
    from paper_2502_19405_amd import repops
    repops.load()
    return repops


def choice(rp, m, n, k, **shape):
    """(kind, index) of REPOPS_LAUNCH_AUTO; one product of dense rows by default."""
    return gemm_choice.choice({"m": m, "n": n, "k": k, "batch": 1, "ta": 0, "tb": 0, "causal": 0,
                               **shape})


def tile(rp, index):
    """Rows, columns and, of a split entry, waves of a matrix-core table entry."""
    name = rp.gemm_configs(rp.LAUNCH_GEMM_MFMA)[index]
    bm, bn = (int(x) for x in name.split("x")[:2])
    waves = re.search(r"/k(\d+)", name)
    return bm, bn, int(waves.group(1)) if waves else None


@pytest.mark.parametrize("m,n,k,batch", [(1, 1, 64, 1 << 24), (1, 1, 256, 1 << 25),
                                         (1 << 30, 4, 4, 1), (1, 1 << 28, 4, 1),
                                         (4, 4, 64, 10_000_000), (16, 16, 128, (1 << 23) + 1),
                                         (16, 16, 128, 1 << 22)])
@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb", [0, 1])
def test_a_split_launch_stays_below_2_to_the_32_threads(rp, m, n, k, batch, ta, tb):
    """One workgroup per tile, and HIP refuses launches of 2^32 threads or more."""
    kind, index = choice(rp, m, n, k, batch=batch, ta=ta, tb=tb)
    assert kind == rp.LAUNCH_GEMM_MFMA
    bm, bn, waves = tile(rp, index)
    if waves:
        assert -(-m // bm) * -(-n // bn) * batch * 64 * waves < 1 << 32


@pytest.mark.parametrize("m,n,k,ld", [(4096, 4096, 64, {"lda": (1 << 22) + 4}),
                                      (4096, 4096, 256, {"ldb": (1 << 22) + 4}),
                                      (128, 1 << 23, 64, {}),          # B's rows
                                      (1 << 23, 128, 128, {"ta": 1}),  # A's columns
                                      (1, 1, 64, {"batch": 1 << 24, "tb": 1})])
def test_short_contractions_the_split_kernels_decline_keep_the_ring_form(rp, m, n, k, ld):
    """Leading dimensions over 2^22, or too many tiles for one workgroup each: with
    at least four tiles of 128 x 128 per compute unit the ring form runs them
    (128 x 8388608 outputs at k 64: 1910 us against 2430 on entry 2)."""
    assert choice(rp, m, n, k, **ld) == (rp.LAUNCH_GEMM_MFMA, 9)
    if "batch" not in ld:  # few tiles: the register-staged form, as for other short k
        few = {"lda": 1 << 23, "ldb": 1 << 23}
        assert choice(rp, 2048, 2048, k, **few) == (rp.LAUNCH_GEMM_MFMA, 2)


def test_the_choice_stays_near_the_fastest_entry():
    """Over the recorded timings of every entry: a change of the estimates (or a new
    file of timings) that sends products to slow entries fails here.  1.04 when this
    was written; a rule by size alone (64 x 64 tiles up to 2^20 outputs,
    else the large tile) is at 3."""
    loss = [us[gemm_choice.choice(s)[1]] / min(us.values())
            for s, us in gemm_choice.recorded(TIMINGS)]
    assert len(loss) > 400
    assert math.exp(sum(math.log(x) for x in loss) / len(loss)) < 1.06


@pytest.mark.parametrize("k", [64, 128, 192, 256])
@pytest.mark.parametrize("tb", [0, 1])
def test_the_ring_form_is_offered_only_where_it_runs(rp, k, tb):
    """Up to one tile per compute unit entry 9's launch is entry 0's kernel, so one
    computation has one price: entry 0's."""
    for m in (128, 256, 384, 512, 768, 1024, 2048):
        for n in (128, 512, 768, 1024, 2048, 4096, 8192):
            for batch in (1, 4, 12, 32):
                for causal in (0, 1) if m == n else (0,):
                    t, u = m // 128, n // 128
                    tiles = (t * (t + 1) // 2 if causal else t * u) * batch
                    s = {"m": m, "n": n, "k": k, "batch": batch, "ta": 0, "tb": tb,
                         "causal": causal}
                    assert (gemm_choice.estimate(s, 9) > 0) == (tiles > gemm_choice.CUS), s


def test_no_recorded_product_is_slower_than_by_size():
    """The estimates never do worse than the rule by size that they replaced: 64 x 64
    tiles up to 2^20 outputs, register-staged slices for k <= 256, 64-row tiles where
    A is zero above its diagonal, else the large tile.  (5%: the spread of a
    recorded time.)"""
    for s, us in gemm_choice.recorded(TIMINGS):
        if s["m"] * s["n"] * s["batch"] <= 1 << 20:
            by_size = 5
        elif s["k"] <= 256:
            by_size = 2
        else:
            by_size = 8 if s["causal"] == 2 else 0
        assert us[gemm_choice.choice(s)[1]] <= 1.05 * us[by_size], s


@pytest.mark.parametrize("k", [(1 << 29) + 64, (1 << 30) + 64, (1 << 31) - 128])
def test_the_staged_kernels_take_any_depth(rp, k):
    """The register-staged kernel that would stand in needs twice the time a block."""
    s = {"m": 256, "n": 256, "k": k, "batch": 1, "ta": 0, "tb": 0, "causal": 0}
    short = {**s, "k": 1 << 20}
    assert gemm_choice.estimate(s, 0) < 1.01 * k / (1 << 20) * gemm_choice.estimate(short, 0)
