"""Exact block attention mass on the GPU (cosa_block_mass) against the oracle's definition."""
import sys

import numpy as np
import pytest

from oracle import cosa_oracle as O
from paper_2607_25291_amd import binding as B
from paper_2607_25291_amd.inputs import WORKLOADS, Workload, make_inputs
from tests.gpu_util import Run, torch

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


SMALL_GQA = Workload("small_gqa", 2, 8, 2, 2048, 128, 128, 16, 0.25, 0.125, 256, (0.005, 0.03))


def gpu_mass(w, q, k):
    p = B.Problem(w.batch, w.n_q_heads, w.n_kv_heads, w.seq_len, w.head_dim, w.block, w.stride)
    run = Run.upload(p, q, k, k)
    nb = w.n_blocks
    out = []
    for _ in range(2):
        m = run._zeros((w.batch, w.n_kv_heads, nb, nb), torch().float32)
        B.cosa_block_mass(p, run.q, run.k, m)
        torch().cuda.synchronize()
        out.append(m.cpu().numpy())
    assert np.array_equal(out[0], out[1]), "block mass is not deterministic"
    return out[0]


@pytest.mark.parametrize("name", ["tiny_l2k", "small_gqa"])
def test_block_mass_full(name):
    w = WORKLOADS["tiny_l2k"] if name == "tiny_l2k" else SMALL_GQA
    say(f"[block mass] {w.name}")
    q, k, v = make_inputs(w)
    G, b = w.n_q_heads // w.n_kv_heads, w.block
    got = gpu_mass(w, q, k)
    ref = O.block_mass(q, k, n_kv_heads=w.n_kv_heads, block=b)
    np.testing.assert_allclose(got, ref, rtol=2e-4, atol=1e-5 * G * b)
    nb = w.n_blocks
    tot = np.array([[[got[n, g, i, :i + 1].sum() for i in range(nb)] for g in range(w.n_kv_heads)]
                    for n in range(w.batch)])
    np.testing.assert_allclose(tot, G * b, rtol=1e-4)
    say(f"  max abs err {np.abs(got - ref).max():.2e} (row block total {G * b})")


def test_block_mass_sampled_32k():
    w = WORKLOADS["qwen3_8b_l32k"]
    say(f"[block mass] {w.name}, sampled units")
    q, k, v = make_inputs(w)
    G, b = w.n_q_heads // w.n_kv_heads, w.block
    got = gpu_mass(w, q, k)
    units = [(0, 0, 0), (0, 3, 130), (0, 7, w.n_blocks - 1)]
    ref = O.block_mass(q, k, n_kv_heads=w.n_kv_heads, block=b, units=units)
    for (n, g, i) in units:
        np.testing.assert_allclose(got[n, g, i, :i + 1], ref[(n, g, i)], rtol=2e-4,
                                   atol=1e-5 * G * b)
        assert abs(got[n, g, i, :i + 1].sum() - G * b) < 1e-4 * G * b


@pytest.mark.parametrize("heads,block,nb,batch", [
    ((1, 1), 64, 1, 1), ((1, 1), 128, 1, 2), ((3, 1), 64, 5, 1), ((6, 2), 64, 3, 2),
    ((10, 2), 128, 3, 1), ((2, 1), 128, 7, 1), ((8, 1), 64, 6, 1), ((12, 3), 128, 4, 1)])
def test_block_mass_head_groups(heads, block, nb, batch):
    """One, two and four query heads per workgroup, one and several passes over the group, both block
    sizes and the first rows of the first block (which see whole tiles of masked keys)."""
    Hq, Hkv = heads
    say(f"[block mass] heads={heads} block={block} nb={nb} batch={batch}")
    w = Workload("m", batch, Hq, Hkv, nb * block, 128, block, block // 8, 0.5, 0.25, 64, 0.02)
    q, k, _ = make_inputs(w)
    got = gpu_mass(w, q, k)
    ref = O.block_mass(q, k, n_kv_heads=Hkv, block=block)
    np.testing.assert_allclose(got, ref, rtol=2e-4, atol=1e-5 * Hq // Hkv * block)


def test_block_mass_most_blocks():
    """The most blocks a call takes (8192): every row's masses sum to the rows of its block, sampled rows
    against float64, and one block more is refused."""
    t = torch()
    nb, b, D = 8192, 64, 128
    say(f"[block mass] most blocks: nb={nb} block={b}")
    gen = t.Generator(device="cuda").manual_seed(1)
    q, k = (t.randn(1, 1, nb * b, D, generator=gen, device="cuda", dtype=t.float32).to(t.bfloat16)
            for _ in range(2))
    mass = t.zeros((1, 1, nb, nb), dtype=t.float32, device="cuda")
    B.cosa_block_mass(B.Problem(1, 1, 1, nb * b, D, b, b // 8), q, k, mass)
    assert bool(((mass.tril().sum(-1) - b).abs() < 1e-4 * b).all())
    for i in (0, 1, 4095, nb - 1):
        x = q[0, 0, i * b:(i + 1) * b].double() @ k[0, 0, :(i + 1) * b].double().T / D ** 0.5
        x[:, i * b:].masked_fill_(t.ones(b, b, dtype=t.bool, device="cuda").triu(1), float("-inf"))
        ref = t.softmax(x, 1).view(b, i + 1, b).sum((0, 2))
        np.testing.assert_allclose(mass[0, 0, i, :i + 1].cpu().numpy(), ref.cpu().numpy(), rtol=2e-4)
    with pytest.raises(B.CosaError) as e:
        B.cosa_block_mass(B.Problem(1, 1, 1, (nb + 1) * b, D, b, b // 8), q, k, mass)
    assert e.value.status == B.COSA_ERR_UNSUPPORTED
