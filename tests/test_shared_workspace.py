"""One transform+quant workspace (or the allocation-free scratch) used in turn
by calls of several shapes: a call leaves the timeout words of every other
shape alone, and the tag of captured calls goes on advancing."""
import numpy as np
import pytest

import paper_2603_04359_amd as cat
from oracle import cat_oracle as o
from paper_2603_04359_amd import binding as B

from gpu_common import check_codes, dev, host, say, torch_mod
from test_gpu_asym import _check_asym
from test_gpu_parity import _rand_T, _wide_X

HEAD = 4096     # bytes at the start of a workspace that hold only these words


def test_timeout_words_lie_in_the_head_of_every_workspace():
    seen = {}
    for d in (256, 2048, 4096, 8192, 14336, 131072):
        for n in list(range(1, 700)) + [1024, 4096, 8192, 16384, 65536]:
            fo = cat.cat_transform_quant_flag_offset(n, d, 128)
            # past the tag word's line, inside the head, a word of its own
            assert 64 <= fo and fo + 4 <= HEAD and fo % 4 == 0, (n, d, fo)
            if d in (2048, 4096, 8192) and n <= 331:
                assert seen.setdefault(fo, (n, d)) == (n, d)
    # the workspace and the scratch hold the head on top of the regions: what
    # fitted the scratch's 16 MiB (with a head of 256 bytes) still does
    for n, d in ((1, 2), (48, 14336), (61680, 4096), (61681, 4096), (8192, 14336), (116508, 2048)):
        regions = 8 * (-(-n // 16) * 16) * (max(1, d // 128) + 1) + 8 * n
        need = cat.cat_transform_quant_workspace_bytes(n, d, 128)
        assert need == regions + HEAD
        assert (need <= B.cat_transform_quant_noalloc_max_bytes()) == (regions + 256 <= 16 << 20)


def _call(X, T, k, ws, asym):
    torch = torch_mod()
    n, d = X.shape
    codes = torch.empty((n, d // 2), dtype=torch.uint8, device="cuda")
    s_x = torch.empty(n, dtype=torch.float32, device="cuda")
    zmin = torch.zeros(n, dtype=torch.float32, device="cuda")

    def run(to=ws):
        if to is None:
            cat.cat_transform_quant_noalloc(X, T, k, codes, s_x)
        elif asym:
            cat.cat_transform_quant_asym(X, T, k, codes, s_x, zmin, to)
        else:
            cat.cat_transform_quant(X, T, k, codes, s_x, to)
    return run, (codes, s_x, zmin)


# a narrow single-pass call, then a call whose words reach over where a word
# placed by the first call's shape would lie: slots, the group kernel's words
# and the exchange words of a wider single pass
@pytest.mark.gpu
@pytest.mark.parametrize("other", [(257, 14336, 256), (100, 14336, 512), (700, 4096, 64), (600, 8192, 128)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_status_of_one_shape_is_left_alone_by_another(other, noalloc):
    say(f"tq shared workspace: 64 x 4096, then {other}, noalloc={noalloc}")
    torch = torch_mod()
    n, d, k = 64, 4096, 128
    X, T = _wide_X(n, d, seed=50), _rand_T(d, k, seed=51)
    Xo, To = _wide_X(other[0], other[1], seed=52), _rand_T(other[1], other[2], seed=53)
    ws = None if noalloc else torch.zeros(
        max(cat.cat_transform_quant_workspace_bytes(n, d, k),
            cat.cat_transform_quant_workspace_bytes(*other)), dtype=torch.uint8, device="cuda")

    def status():
        if noalloc:
            cat.cat_transform_quant_noalloc_status(n, d, k)
        else:
            cat.cat_transform_quant_status(ws, n, d, k)

    if noalloc:
        try:
            status()
        except cat.CatError:
            pass                      # cleared: whatever earlier calls left
    run, (codes, s_x, _) = _call(dev(X, "bf16"), dev(T, "bf16"), k, ws, False)
    other_run, (codes_o, _, _) = _call(dev(Xo, "bf16"), dev(To, "bf16"), other[2], ws, False)
    run()
    other_run()
    status()                          # no wait ran out
    check_codes(host(codes), X, T, label="first shape")
    check_codes(host(codes_o), Xo, To, label="other shape")
    if not noalloc:
        # a word that reports a timeout stays set, also over rows of zeros
        fo = cat.cat_transform_quant_flag_offset(n, d, k)
        ws[fo:fo + 4].fill_(1)
        zero_run, _ = _call(torch.zeros(other[:2], dtype=torch.bfloat16, device="cuda"),
                            dev(To, "bf16"), other[2], ws, False)
        zero_run()
        with pytest.raises(cat.CatError) as e:
            status()
        assert e.value.code == cat.CAT_ERR_TIMEOUT
        status()


@pytest.mark.gpu
@pytest.mark.parametrize("asym", [True, False])
def test_replays_of_two_shapes_on_one_workspace(asym):
    # a graph of a single-pass call and a two-pass call with zero rows: the
    # rows' keys are the same on every replay, so a tag word that they
    # overwrote would start from the same value each time
    say(f"tq graph of two shapes on one workspace, asym={asym}")
    torch = torch_mod()
    shapes = [(48, 4096, 128), (48, 14336, 256)]
    size = cat.cat_transform_quant_asym_workspace_bytes if asym else cat.cat_transform_quant_workspace_bytes
    ws = torch.zeros(max(size(*s) for s in shapes), dtype=torch.uint8, device="cuda")
    own = torch.zeros_like(ws)
    Ts = [_rand_T(d, k, seed=54 + i) for i, (n, d, k) in enumerate(shapes)]
    Xd = [torch.zeros((n, d), dtype=torch.bfloat16, device="cuda") for n, d, k in shapes]
    calls = [_call(Xd[i], dev(Ts[i], "bf16"), shapes[i][2], ws, asym) for i in range(2)]
    for run, _ in calls:
        run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        for run, _ in calls:
            run()
    for rep in range(6):
        Xs = [_wide_X(n, d, seed=60 + 2 * rep + i) * 2.0 ** -rep for i, (n, d, k) in enumerate(shapes)]
        Xs[1][::2] = 0.0              # padded tokens
        for i in range(2):
            Xd[i].copy_(dev(Xs[i], "bf16"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = [[host(v).copy() for v in out] for _, out in calls]
        # eager calls on a workspace of their own give the same bits
        for i, (run, out) in enumerate(calls):
            own.zero_()
            run(own)
            assert all(np.array_equal(a, host(b)) for a, b in zip(got[i], out)), f"replay {rep}, call {i}"
        if rep in (0, 5):
            for i in range(2):
                c, s, z = got[i]
                if asym:
                    _check_asym(o.unpack_int4(c).astype(np.int16) + 8, s, z, Xs[i], Ts[i],
                                f"replay {rep}, call {i}")
                else:
                    check_codes(c, Xs[i], Ts[i], label=f"replay {rep}, call {i}")
        cat.cat_transform_quant_status(ws, *shapes[0])


# every two-pass route: slots, wide, group, ring, whole-key vector ALU, mfma
@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k,dtype", [
    (257, 14336, 256, "bf16"), (3000, 14336, 128, "bf16"), (300, 4096, 64, "bf16"), (64, 1024, 512, "bf16"),
    (100, 640, 128, "bf16"), (100, 96, 32, "bf16"), (30, 4352, 64, "f32"), (40, 64, 8, "f32")])
@pytest.mark.parametrize("asym", [True, False])
def test_two_pass_words_carry_no_tag(n, d, k, dtype, asym):
    # a single-pass call of another shape on the workspace takes a 64-bit word
    # whose upper half is its tag (bit 31 set) for a published one
    say(f"tq two-pass words {n} x {d}, k={k} {dtype} asym={asym}")
    torch = torch_mod()
    size = cat.cat_transform_quant_asym_workspace_bytes if asym else cat.cat_transform_quant_workspace_bytes
    ws = torch.zeros(size(n, d, k), dtype=torch.uint8, device="cuda")
    run, _ = _call(dev(_wide_X(n, d, seed=70), dtype), dev(_rand_T(d, k, seed=71), dtype), k, ws, asym)
    run()
    words = host(ws)
    assert not words[:HEAD].any()
    assert (words[HEAD:].view(np.int64) >= 0).all()
