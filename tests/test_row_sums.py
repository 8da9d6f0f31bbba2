"""The FP32 sums of a server's row kernels: no longer, and no less exact, than the
72-pair tiles of the block kernels (and of the pair kernels of large problems).

The two orders of summation are emulated on the CPU over the same FP32 terms (the
kernels' products, without fused multiply-adds) and compared with the same sums in
64 bits.  Rows: a lane adds every 64th pair of its wave's tiles, the sums of four
lanes are added in FP32, the rest in FP64; A1 / kappa and -A2 share a sum, with p_j /
kappa rounded.  Blocks: a lane adds its landmark's pairs, 72 at a time."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KAPPA = 2.0 * np.log(2.0)
F = np.float32


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = tmp_path_factory.mktemp("plan") / "batch_plan_dump"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1907_04839_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "batch_plan_dump.cpp"), "-o", str(exe)],
                   check=True)

    def of(*sizes):
        out = subprocess.run([str(exe), *map(str, sizes)], capture_output=True, text=True, check=True)
        return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    return of


def test_a_served_fp32_sum_covers_72_pairs_at_most(plan):
    for n, _, _, pairs, tile in plan(1, 64, 65, 1000, 4607, 4608, 4609, 8191, 8192, 9217, 16383,
                                     16384, 65536):
        assert tile == 72 and pairs <= tile, (n, pairs)


def test_a_row_plans_fp32_sum_covers_72_pairs_at_most(tmp_path):
    exe = tmp_path / "row_pairs_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1907_04839_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "row_pairs_test.cpp"), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "row pairs ok" in out.stdout, out.stdout


def row_sums(terms, jg, round_):
    """Sums over axis 1 of the terms ([rows, n] each, added one after the other)."""
    rows, n = terms[0].shape
    nt = (n + 63) // 64
    tiles = []
    for x in terms:
        t = np.zeros((rows, nt * 64), F)
        t[:, :n] = x
        tiles.append(t.reshape(rows, nt, 64))
    total = np.zeros(rows)
    for w in range(jg):
        for t0 in range(w, nt, round_ * jg):
            h = np.zeros((rows, 64), F)
            for t in range(t0, min(nt, t0 + round_ * jg), jg):
                for x in tiles:
                    h = h + x[:, t]
            h = h[:, :32] + h[:, 32:]
            total += (h[:, :16] + h[:, 16:]).astype(np.float64).sum(1)
    return total


def block_sums(term, waves=12, tile=72):
    rows, n = term.shape
    chunk = -(-n // waves)
    total = np.zeros(rows)
    for c0 in range(0, n, chunk):
        c1 = min(n, c0 + chunk)
        for a in range(c0, c1, tile):
            h = np.zeros(rows, F)
            for j in range(a, min(c1, a + tile)):
                h = h + term[:, j]
            total += h
    return total


def pair_terms(rec, idx, dtype):
    """Per pair of a row of idx: g p_j (forward), g s db (A1), g (pi + s e) D (A2)."""
    q, p, a, b = (x.astype(dtype) for x in rec)
    d, ex = q[idx][:, None] - q[None], b[idx][:, None] - b[None]
    g = np.exp2(-(d * d).sum(2))
    dot = lambda x, y: (x[idx][:, None] * y[None]).sum(2)   # noqa: E731
    s = dot(p, p)
    v = dot(a, p) + dot(p, a) + s * (d * ex).sum(2)
    s_scaled = dot(p, (p * dtype(1.0 / KAPPA)).astype(dtype))
    return (g[..., None] * p[None], (g * s)[..., None] * ex, (g * v)[..., None] * d,
            (g * s_scaled)[..., None] * ex)


def errors(n, seed, jg, round_, rows=24):
    """rms errors (blocks, rows) of the forward sum and of A1 / kappa - A2."""
    rng = np.random.default_rng(seed)
    q, p = 15.0 * rng.normal(size=(n, 3)), 0.5 * rng.normal(size=(n, 3))
    a, b = rng.normal(size=(n, 3)), rng.normal(size=(n, 3))
    k = np.sqrt(0.5 * np.log2(np.e)) / 6.0
    rec = [x.astype(F) for x in (k * q, p, a, KAPPA * k * b)]
    idx = rng.choice(n, rows, replace=False)
    h64, a164, a264, _ = pair_terms(rec, idx, np.float64)
    h, a1, a2, a1k = pair_terms(rec, idx, F)
    assert h.dtype == a1k.dtype == F
    e = np.zeros((2, 2))
    for c in range(3):
        ref = (h64[:, :, c].sum(1), a164[:, :, c].sum(1) / KAPPA - a264[:, :, c].sum(1))
        blocks = (block_sums(h[:, :, c]),
                  block_sums(a1[:, :, c]) / KAPPA - block_sums(a2[:, :, c]))
        row = (row_sums([h[:, :, c]], jg, round_), row_sums([a1k[:, :, c], -a2[:, :, c]], jg, round_))
        for kind, got in enumerate((blocks, row)):
            e[kind] += [np.square(x - r).sum() for x, r in zip(got, ref)]
    return e


@pytest.mark.parametrize("n", [8000, 9300, 16000, 20000, 32000])
def test_row_sums_are_no_less_exact_than_block_sums(plan, n):
    (_, jg, round_, _, _), = plan(n)
    blocks, rows = np.sqrt(sum(errors(n, seed, jg, round_) for seed in range(3)))
    print(f"[n={n} jg={jg} round={round_}] forward {rows[0] / blocks[0]:.2f}, "
          f"A {rows[1] / blocks[1]:.2f} of the blocks' rms error")
    assert rows[0] <= blocks[0] and rows[1] <= blocks[1]
