"""GPU parity of the tensor commitment (repops_commit) against the CPU oracle:
byte-identical 32-byte digests for every size class (empty, one byte, one
chunk, chunk +- 1, odd and power-of-two leaf counts, trees deeper than the
single-workgroup top), unaligned data and chunk sizes off the vector path, and
model-sized tensors."""
import numpy as np
import pytest

import oracle
from gpu_util import announce, dev, host
from paper_2502_19405_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2502_19405_amd import repops
    repops.load()
    return repops


def gpu_commit(rp, buf_u8, chunk):
    """Digest of a uint8 host buffer, placed at the start of a device tensor."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(buf_u8)).to("cuda:0")
    return bytes(host(rp.commit(t, chunk)).tobytes())


@pytest.mark.parametrize("chunk", [64, 1024, 4096, 100])
def test_commit_sizes(rp, chunk):
    g = inputs.rng(950 + chunk)
    # leaf counts around the 256 leaves one workgroup reduces, and (64-byte
    # chunks) more than 512 x 256 leaves, so a level launch runs as well
    sizes = [0, 1, 3, 63, 64, 65, chunk - 1, chunk, chunk + 1, 2 * chunk, 3 * chunk + 7,
             255 * chunk, 256 * chunk, 257 * chunk + 5, 513 * chunk, 512 * chunk,
             1025 * chunk - 3, 5000 * chunk + 1]
    if chunk == 64:
        sizes.append((512 * 256 + 300) * chunk + 9)
    for n in sizes:
        if n < 0:
            continue
        data = g.integers(0, 256, n).astype(np.uint8)
        announce("commit", chunk, n)
        assert gpu_commit(rp, data, chunk) == oracle.commit(data, chunk), (chunk, n)


def test_commit_unaligned_views(rp):
    import torch
    g = inputs.rng(951)
    data = g.integers(0, 256, 70001).astype(np.uint8)
    base = torch.from_numpy(data).to("cuda:0")
    for off in (1, 2, 3, 4, 8, 12, 16):
        announce("commit unaligned", off)
        view = base[off:]
        got = bytes(host(rp.commit(view, 1024)).tobytes())
        assert got == oracle.commit(data[off:], 1024), off


def test_commit_float_tensors(rp):
    g = inputs.rng(952)
    for shape in ((768, 3072), (4096, 768), (1000, 999)):
        X = inputs.normal(g, shape)
        announce("commit tensor", shape)
        got = bytes(host(rp.commit(dev(X), 1024)).tobytes())
        assert got == oracle.commit(X, 1024), shape


def test_commit_llama_mlp_weight(rp):
    """A Llama-8B feed-forward weight, 4096 x 14336 fp32 (235 MB, 229376
    leaves, 18 tree levels)."""
    g = inputs.rng(953)
    W = inputs.normal(g, (4096, 14336), var=4e-4)
    announce("commit llama weight")
    got = bytes(host(rp.commit(dev(W), 1024)).tobytes())
    assert got == oracle.commit(W, 1024)


@pytest.mark.parametrize("leaves", [127, 128, 129, 256, 257, 384, 512, 513, 16384, 16385,
                                    16640, 32768, 32769, 65536, 65537])
@pytest.mark.parametrize("short", [0, 3])
def test_commit_launch_edges(rp, leaves, short):
    """Leaf counts where the launches change: 128 leaves to a workgroup of two
    waves a leaf, up to 32768 of them; 256 nodes to a tree slice, over 16384 and up
    to 65536 of them in slices; with a whole and a short last chunk."""
    data = inputs.rng(954 + leaves).integers(0, 256, leaves * 64 - short).astype(np.uint8)
    announce("commit launches", leaves, short)
    assert gpu_commit(rp, data, 64) == oracle.commit(data, 64)


# tensors shorter than their chunk, alone or as the only leaf of a last workgroup
# of 128 leaves (whole leaves before it), up to the largest chunk accepted
@pytest.mark.parametrize("nbytes,chunk", [(1, 64), (100, 128), (100, 1 << 20), (4100, 1 << 20),
                                          (100, 1 << 30), (128 * 4096 + 100, 4096),
                                          (2 * 128 * 1024 + 1, 1024), (1 << 20, (1 << 20) + 64)])
def test_commit_short_leaf_alone(rp, nbytes, chunk):
    data = inputs.rng(955 + nbytes).integers(0, 256, nbytes).astype(np.uint8)
    announce("commit short leaf", nbytes, chunk)
    assert gpu_commit(rp, data, chunk) == oracle.commit(data, chunk)


def test_commit_costs_its_bytes_not_its_chunk(rp):
    """100 bytes take one leaf and no level whatever the chunk: the time with
    1 MiB chunks is that with 128-byte ones.  (Walking the 16385 blocks of a 1 MiB
    chunk with four barriers each takes over a hundred times as long; the factor 4
    leaves room for the clock.)"""
    import torch
    t = dev(inputs.rng(956).integers(0, 256, 100).astype(np.uint8))

    def us(chunk):
        ws = torch.empty(64, dtype=torch.int32, device="cuda:0")
        digest = torch.empty(32, dtype=torch.uint8, device="cuda:0")
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                rp.commit(t, chunk, digest=digest, workspace=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / 20)
        return best

    announce("commit short leaf time")
    us(128)
    assert us(1 << 20) < 4 * us(128)
