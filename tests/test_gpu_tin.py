"""GPU parity of the generated index-notation leaves (spl_tin_*) against the
general oracle (oracle/tin.py): CSR output patterns bit for bit, values
within 1e-12 S (FP64) or 1e-5 S (FP32) on sampled rows of the outermost index
(600 rows: three workgroups and a ragged tail), small-integer values bit for
bit, every dense output entry written, and repeated calls identical."""
import numpy as np
import pytest
import torch

from oracle import tin as T
from tests.gpu_util import RTOL, assert_close, host64, need_gpu
from tests.tin_cases import CASES, EXTENTS, SMALL, make

pytestmark = pytest.mark.gpu


def _spl():
    need_gpu()
    import paper_2207_13901_amd as spl
    return spl


def _rows(n, three_level):
    rs = np.random.RandomState(n)
    k = 12 if three_level else 40
    return np.unique(np.concatenate([[0, 1, 2, 3, 7, 255, 256, n - 1],
                                     rs.choice(n, k, replace=False)]))


def _run(spl, stmt, kind, lib, shape, dtype, dev):
    if kind == "csr":
        return spl.tin(stmt, shape=shape, **lib)
    if kind == "scalar":
        return spl.tin(stmt, **lib)
    out = torch.full(shape, float("nan"), dtype=dtype, device=dev)
    return spl.tin(stmt, out, **lib)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]} [{c[1]}]" for c in CASES])
def test_tin_matches_oracle(case, dtype):
    spl = _spl()
    stmt, kind, recipe = case
    dev = torch.device("cuda", 0)
    ext = SMALL if kind == "scalar" else EXTENTS
    lib, ref, shape = make(stmt, recipe, dtype, seed=11, extents=ext, device=dev)
    print(f"tin: {stmt} [{kind}] {dtype}", flush=True)
    got = _run(spl, stmt, kind, lib, shape, dtype, dev)
    torch.cuda.synchronize()
    rtol = RTOL[dtype]
    if kind == "scalar":
        want, S = T.evaluate(stmt, ref)
        assert_close(host64(got), np.reshape(want, 1), np.reshape(S, 1), rtol, stmt)
        return
    three = any(v == "csf" or v == "ddc" for v in recipe.values())
    rows = _rows(shape[0], three)
    want, S = T.evaluate(stmt, ref, out_shape=shape, rows=rows)
    if kind == "csr":
        pos, crd = T.pattern(stmt, ref, shape)
        assert np.array_equal(got.pos.cpu().numpy(), pos), stmt
        assert np.array_equal(got.crd.cpu().numpy(), crd), stmt
        vals = host64(got.vals)
        for r, i in enumerate(rows):
            cols = crd[pos[i]:pos[i + 1]]
            assert_close(vals[pos[i]:pos[i + 1]], want[r, cols], S[r, cols], rtol,
                         f"{stmt} row {i}")
        return
    host = host64(got)
    assert not np.isnan(host).any(), "every output entry is written"
    assert_close(host[rows], want, S, rtol, stmt)


@pytest.mark.parametrize("case", [c for c in CASES if c[1] != "scalar"],
                         ids=[f"{c[0]} [{c[1]}]" for c in CASES if c[1] != "scalar"])
def test_tin_integer_values_bit_exact_and_deterministic(case):
    spl = _spl()
    stmt, kind, recipe = case
    dev = torch.device("cuda", 0)
    lib, ref, shape = make(stmt, recipe, torch.float64, seed=12, kind="int", extents=EXTENTS,
                           device=dev)
    got = _run(spl, stmt, kind, lib, shape, torch.float64, dev)
    again = _run(spl, stmt, kind, lib, shape, torch.float64, dev)
    three = any(v == "csf" or v == "ddc" for v in recipe.values())
    rows = _rows(shape[0], three)
    want, _ = T.evaluate(stmt, ref, out_shape=shape, rows=rows)
    if kind == "csr":
        assert torch.equal(got.vals, again.vals) and torch.equal(got.crd, again.crd)
        pos = got.pos.cpu().numpy()
        crd = got.crd.cpu().numpy()
        vals = host64(got.vals)
        for r, i in enumerate(rows):
            assert np.array_equal(vals[pos[i]:pos[i + 1]], want[r, crd[pos[i]:pos[i + 1]]]), i
        return
    assert torch.equal(got, again)
    assert np.array_equal(host64(got)[rows], want), stmt


def test_tin_scalar_on_a_larger_pattern():
    # the co-iterated 2-D inner product over 600 rows (three workgroups of
    # partials and the fixed-order final sum)
    spl = _spl()
    stmt = "a = B(i,j) * C(i,j)"
    dev = torch.device("cuda", 0)
    lib, ref, _ = make(stmt, dict(B="csr", C="csr"), torch.float64, seed=13, extents=EXTENTS,
                       device=dev)
    got = spl.tin(stmt, **lib)
    want, S = T.evaluate(stmt, ref)
    assert_close(host64(got), np.reshape(want, 1), np.reshape(S, 1), 1e-12, stmt)


# CSR outputs of CSR operands: the workgroups' rows staged in LDS, and in the
# same launch a row too long for the stage (entries of 20 times the mean)
@pytest.mark.parametrize("n,m,deg,long", [(1, 1, 1, ()), (128, 700, 3, ()), (129, 700, 3, ()),
                                          (700, 9000, 2, (0, 130, 699)), (1000, 400, 60, ()),
                                          (300, 3000, 900, ()), (257, 50, 0, (200,))])
@pytest.mark.parametrize("stmt", ["A(i,j) = B(i,j) - C(i,j)", "A(i,j) = B(i,j) * C(i,j)",
                                  "A(i,j) = B(i,j) * c(j) - C(i,j) * d(i)"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_tin_csr_outputs_staged_and_direct_rows(n, m, deg, long, stmt, dtype):
    spl = _spl()
    dev = torch.device("cuda", 0)
    rs = np.random.RandomState(n + m)
    print(f"tin staged: {stmt} n={n} m={m} deg={deg} {dtype}", flush=True)

    def operand():
        dense = np.where(rs.rand(n, m) < deg / m, rs.uniform(-1, 1, (n, m)), 0.0)
        for i in long:
            dense[i] = rs.uniform(0.5, 1, m)
        dense = torch.as_tensor(dense).to(dtype)
        mask = dense != 0
        pos = torch.zeros(n + 1, dtype=torch.int32)
        pos[1:] = mask.sum(1).cumsum(0)
        crd = mask.nonzero()[:, 1].to(torch.int32)
        return dense.double(), mask, spl.CSR(pos.to(dev), crd.to(dev), dense[mask].to(dev), (n, m))

    (Bd, Bm, B), (Cd, Cm, C) = operand(), operand()
    c, d = (torch.as_tensor(rs.uniform(-1, 1, k)).to(dtype) for k in (m, n))
    args = dict(B=B, C=C)
    if "*" not in stmt:
        want, S, mask = Bd - Cd, Bd.abs() + Cd.abs(), Bm | Cm
    elif "c(j)" not in stmt:
        want, S, mask = Bd * Cd, (Bd * Cd).abs(), Bm & Cm
    else:
        args.update(c=c.to(dev), d=d.to(dev))
        tb, tc = Bd * c.double(), Cd * d.double()[:, None]
        want, S, mask = tb - tc, tb.abs() + tc.abs(), Bm | Cm
    A = spl.tin(stmt, shape=(n, m), **args)
    pos = np.concatenate([[0], mask.sum(1).cumsum(0).numpy()])
    assert np.array_equal(A.pos.cpu().numpy(), pos)
    assert np.array_equal(A.crd.cpu().numpy(), mask.nonzero()[:, 1].numpy())
    assert_close(host64(A.vals), want[mask].numpy(), S[mask].numpy(), RTOL[dtype], stmt)


# The scan of the row counts: one tile, a remainder, and either side of the
# tiles whose sums the last step adds up by itself.
@pytest.mark.parametrize("n", [1, 4096, 4097, 4096 * 4096, 4096 * 4096 + 1])
def test_csr_output_positions(n):
    spl, dev = _spl(), torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(n % 1000)
    m = 50
    keys = [torch.unique(torch.randint(0, n * m, (3000,), generator=g, device=dev)) for _ in range(2)]
    rows = torch.arange(n + 1, device=dev) * m

    def csr(k):
        return spl.CSR(torch.searchsorted(k, rows).to(torch.int32), (k % m).to(torch.int32),
                       torch.ones(k.numel(), dtype=torch.float64, device=dev), (n, m))

    A = spl.tin("A(i,j) = B(i,j) - C(i,j)", shape=(n, m), B=csr(keys[0]), C=csr(keys[1]))
    union = torch.unique(torch.cat(keys))
    assert torch.equal(A.pos, torch.searchsorted(union, rows).to(torch.int32))
    assert torch.equal(A.crd, (union % m).to(torch.int32))
