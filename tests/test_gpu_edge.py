"""The edge-handling matrix-core kernels (any size, stride, alignment) against the fp64 oracle at the sizes
where they can go wrong: one off the 32 / 64 / 128 tile sides, one element, remainders of a 16-byte vector in
every extent, contractions that are split over workgroups, operands off 16-byte alignment.  Tolerances are
the dtype's (sums of up to a few thousand terms in fp32, one bf16 rounding per intermediate)."""
import numpy as np
import pytest
import torch

from oracle import poetx_oracle as orc
from workloads import round_bf16, round_f32
from tests.harness import TOL, build_blocks, rel_err, run_layer, tdtype, to_dev, to_np
from tests.test_gpu_parity import check_layer, synth_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,n,N,b,k", [
    (8, 8, 1, 8, 2),            # a single token, a block smaller than any tile
    (33, 40, 31, 32, 2),        # one past a block, token remainder 7 of 8
    (96, 65, 33, 32, 3),        # tail blocks of 1 on one side
    (127, 129, 63, 64, 2),      # one off the 128 tile
    (160, 96, 65, 64, 2),
    (1000, 24, 129, 24, 2),     # block side that no tile divides, long contraction split over workgroups
    (72, 2050, 17, 72, 2),      # the same in the backward direction
    (640, 1376, 2047, 64, 2),   # 128-wide tiles, every extent ragged
    (512, 256, 1000, 256, 2),   # large blocks, token count a multiple of 8 only
    # 64-wide tiles whose waves split the stages (fp32 backward), split over workgroups as well.  (A tail block of side 2 would have
    # one parameter: its gradient, one sum of rounded products, has no bound relative to itself where they cancel.)
    (768, 1096, 1001, 64, 2),
    (2000, 2040, 2001, 40, 1),  # 128-wide ones with four waves (bf16 forward) and eight (backward)
    # bf16 rows shorter than a vector, whole vectors, and tails (each loaded in its own way); blocks that no tile divides
    (192, 288, 7, 96, 2),
    (192, 288, 8, 96, 2),
    (192, 288, 9, 96, 2),
    (256, 128, 1041, 64, 2),    # tails behind whole tiles
    (2592, 1950, 33, 64, 3),    # 72 blocks: the sides' series backward in stripes each, in whole blocks together
    (256, 384, 512, 128, 2),    # every tile and stage whole, and all but the last: the block gradients of 520 tokens
    (256, 384, 520, 128, 2),
    # other tiles and splits that the rule gives
    (1032, 1024, 8704, 128, 1), # block gradients on 128 x 128 that fill the chip, of which one side's tiles are whole: each side on its own kernel
    (200, 776, 1001, 40, 1),    # fp32 forward: 64 x 64 with sixteen waves ...
    (1000, 632, 200, 40, 1),    # ... in 6 ranges
    (992, 632, 200, 40, 1),     # a contraction of 16 more takes slices
    (776, 1064, 200, 24, 1),    # fp32 backward: 64 x 64 in 9
    (848, 200, 200, 40, 1),     # bf16 forward: 64 x 64 in 7
    (200, 848, 200, 40, 1),     # ... backward
    (2080, 2048, 24, 32, 1),    # a few tokens of a large weight: slices, ...
    (2100, 2040, 24, 60, 1),    # ... and what they do not take (contractions in no whole slices): splits by workgroups per CU
])
def test_layer_at_tile_edges(lib, m, n, N, b, k, dtype):
    data = synth_layer(9000 + m + n + N + b, m, n, N, b, k, dtype, 0.01)
    ref = orc.linear_fwd_bwd_from_theta(data["X"], data["dZ"], data["W"], data["pi_R"], data["pi_P"],
                                        data["theta_R"], data["theta_P"], b, k)
    check_layer(run_layer(data, dtype), ref, data["pi_P"], dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,b,cols,off", [(64, 32, 96, 1), (256, 256, 256, 1), (320, 64, 40, 3),
                                          (1032, 8, 1021, 1), (2048, 16, 1021, 3)])   # blocks up to 16, 4128 and 4096 tiles: plain kernel
def test_apply_off_alignment(lib, d, b, cols, off, dtype):
    """Input, output and blocks that start `off` elements into an allocation: element alignment is enough, and
    nothing outside the output is written."""
    rng = np.random.Generator(np.random.PCG64(9100 + d + cols))
    V = (round_f32 if dtype == "f32" else round_bf16)(rng.standard_normal((d, cols)))
    E = round_bf16(rng.standard_normal((d // b, b, b)) * 0.05)
    pi = rng.permutation(d).astype(np.int32)
    eye = np.eye(b)
    stored = E + eye if dtype == "f32" else np.stack([E, np.swapaxes(E, 1, 2)], axis=1)
    dt = tdtype(dtype)

    def shifted(a):
        flat = torch.zeros(a.size + off, dtype=dt, device="cuda")
        flat[off:] = to_dev(a, dt).reshape(-1)
        return flat[off:].view(a.shape)
    buf = torch.full((d * cols + 2 * off + 8,), -7.0, dtype=dt, device="cuda")
    out = buf[off:off + d * cols].view(d, cols)
    blocks, Vd = shifted(stored), shifted(V)
    for trans in (False, True):
        lib.poetx_perm_blockdiag_apply_left(Vd, out, torch.from_numpy(pi).cuda(), blocks, b, trans)
        torch.cuda.synchronize()
        assert rel_err(to_np(out), orc.apply_left(V, pi, E + eye, trans)) <= TOL[dtype]
        assert torch.all(buf[:off] == -7.0) and torch.all(buf[off + d * cols:] == -7.0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,n,N,b", [
    (8, 12, 1, 4),              # one token
    (65, 40, 31, 32),           # tail blocks, one off a tile
    (1000, 264, 33, 24),
    (512, 768, 7, 256),         # a contraction of four stages and more per tile
    (1024, 512, 200, 64),       # several token tiles, remainder
])
def test_forward_reads_tokens_in_place(lib, m, n, N, b, dtype):
    """A few token-major tokens are read and written without transposing passes: Z and the saved B are the feature-major
    call's bit for bit, feature-major being checked against the oracle, and nothing outside Z is written."""
    data = synth_layer(9050 + m + n + N, m, n, N, b, 3, dtype, 0.01)
    ref = orc.linear_fwd_bwd_from_theta(data["X"], data["dZ"], data["W"], data["pi_R"], data["pi_P"],
                                        data["theta_R"], data["theta_P"], b, 3)
    res = run_layer(data, dtype)
    # on the tensor's scale: a row of one token may be a sum that cancels, whose error is the dtype's rounding of the terms
    assert rel_err(res["Z"], ref["Z"]) <= TOL[dtype]
    dev = res["dev"]
    desc = lib.make_desc(m, n, b, 3, N, lib.F32 if dtype == "f32" else lib.BF16, layout=lib.TOKEN_MAJOR)
    buf = torch.full((N * n + 16,), -7.0, dtype=tdtype(dtype), device="cuda")
    Zt = buf[8:8 + N * n].view(N, n)
    B = torch.full_like(dev["B"], float("nan"))
    ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4 + 1,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
    lib.poetx_linear_fwd(desc, dev["X"].t().contiguous(), dev["W"], dev["pi_R"], dev["pi_P"], dev["blk_R"], dev["blk_P"], Zt, B, ws)
    torch.cuda.synchronize()
    assert torch.equal(Zt, dev["Z"].t()) and torch.equal(B, dev["B"])
    assert torch.all(buf[:8] == -7.0) and torch.all(buf[8 + N * n:] == -7.0)


@pytest.mark.parametrize("b", [2, 15, 16, 31, 33, 64, 65, 128])
@pytest.mark.parametrize("k", [1, 2, 5])
def test_small_block_series(lib, b, k):
    """The one-launch fp32 series (block sides up to 128, padded to 32 / 64 / 128 on chip): build and backward against
    the oracle in fp32 accuracy (sums of at most 128 k fp32 terms), ragged last block with loud dead slots, accumulate."""
    d = 2 * b + b // 2 + 1 if b > 2 else 5
    rng = np.random.Generator(np.random.PCG64(9200 + b + k))
    nb, L = orc.n_blocks(d, b), b * (b - 1) // 2
    theta = round_f32(rng.standard_normal((nb, L)) * 0.02)
    r = orc.tail_side(d, b)
    iu, ju = np.triu_indices(b, k=1)
    dead = (iu >= r) | (ju >= r)
    theta[-1, dead] = 9.0
    th = to_dev(theta, torch.float32)
    G = torch.empty((nb, b, b), dtype=torch.float32, device="cuda")
    E = torch.empty((nb, 2, b, b), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(lib.poetx_cnp_workspace_bytes(d, b), lib.poetx_cnp_bwd_workspace_bytes(d, b, k)), dtype=torch.uint8, device="cuda")
    lib.poetx_cnp_build(th, d, b, k, lib.CNP_FP32, G, E, ws)
    Q = orc.skew_from_packed(theta, b, d)
    ref = orc.cnp(Q, k)
    eye = np.eye(b)
    assert rel_err(to_np(G) - eye, ref - eye) <= 1e-5
    assert rel_err(to_np(E)[:, 0], ref - eye) <= 2.0 ** -8
    assert torch.equal(E[:, 1], E[:, 0].transpose(1, 2))
    assert np.array_equal(to_np(G)[-1, r:], np.eye(b)[r:]) and np.array_equal(to_np(G)[-1, :, r:], np.eye(b)[:, r:])
    dG = round_f32(rng.standard_normal((nb, b, b)))
    want = orc.packed_from_skew_grad(orc.cnp_bwd(Q, dG, k), b, d)
    for acc, start in ((False, float("nan")), (True, 1.0)):
        dth = torch.full_like(th, start)
        lib.poetx_cnp_bwd(th, to_dev(dG, torch.float32), d, b, k, lib.CNP_FP32, dth, acc, ws)
        got = to_np(dth) - (1.0 if acc else 0.0)
        assert rel_err(got, want) <= 1e-5
        assert np.all(got[-1, dead] == 0)


@pytest.mark.parametrize("b,nb,k", [
    # the last count in column stripes and the first of whole blocks: backward ...
    (64, 64, 4), (64, 65, 4), (48, 85, 2), (48, 86, 2), (128, 64, 3), (128, 65, 3), (100, 73, 1), (100, 74, 1),
    # ... build (below three powers, and from three on)
    (64, 96, 2), (64, 97, 2), (64, 160, 3), (64, 161, 3), (128, 32, 2), (128, 33, 2), (32, 192, 1), (32, 193, 1), (32, 320, 5), (32, 321, 5),
])
def test_small_block_series_of_many_blocks(lib, b, nb, k):
    """Both forms of the one-launch fp32 series on either side of the block counts where it changes from one to the other: first, middle
    and ragged last block against the oracle in fp32 accuracy (sums of at most 128 k fp32 terms), dead slots, accumulate.  Blocks have
    the bits that they have alone; packed gradients too, up to a side of 32, where the backward has one form."""
    r, L = b // 2 + 1, b * (b - 1) // 2
    d = (nb - 1) * b + r
    rng = np.random.Generator(np.random.PCG64(9700 + b + nb + k))
    theta = round_f32(rng.standard_normal((nb, L)) * 0.02)
    iu, ju = np.triu_indices(b, k=1)
    dead = (iu >= r) | (ju >= r)
    theta[-1, dead] = 9.0
    dG = round_f32(rng.standard_normal((nb, b, b)))

    def run(lo, acc, start):
        n, dd = nb - lo, d - lo * b
        th = to_dev(theta[lo:], torch.float32)
        G = torch.full((n, b, b), float("nan"), dtype=torch.float32, device="cuda")
        E = torch.full((n, 2, b, b), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(max(lib.poetx_cnp_workspace_bytes(dd, b), lib.poetx_cnp_bwd_workspace_bytes(dd, b, k)), dtype=torch.uint8, device="cuda")
        lib.poetx_cnp_build(th, dd, b, k, lib.CNP_FP32, G, E, ws)
        dth = torch.full_like(th, start)
        lib.poetx_cnp_bwd(th, to_dev(dG[lo:], torch.float32), dd, b, k, lib.CNP_FP32, dth, acc, ws)
        torch.cuda.synchronize()
        return G, E, dth
    G, E, dth = run(0, False, float("nan"))
    added = to_np(run(0, True, 1.0)[2]) - 1.0
    eye = np.eye(b)
    for at, side in (([0, nb // 2], b), ([nb - 1], r)):
        span = (len(at) - 1) * b + side
        Q = orc.skew_from_packed(theta[at], b, span)
        ref = orc.cnp(Q, k) - eye
        assert rel_err(to_np(G[at]) - eye, ref) <= 1e-5
        assert rel_err(to_np(E[at])[:, 0], ref) <= 2.0 ** -8
        want = orc.packed_from_skew_grad(orc.cnp_bwd(Q, dG[at], k), b, span)
        assert rel_err(to_np(dth[at]), want) <= 1e-5 and rel_err(added[at], want) <= 1e-5
    assert torch.equal(E[:, 1], E[:, 0].transpose(1, 2))
    assert bool(torch.isfinite(dth).all()) and np.all(to_np(dth)[-1, dead] == 0) and np.all(added[-1, dead] == 0)
    G2, E2, dth2 = run(nb - 2, False, float("nan"))
    assert torch.equal(G2, G[-2:]) and torch.equal(E2, E[-2:])
    assert b > 32 or torch.equal(dth2, dth[-2:])


@pytest.mark.parametrize("m,n,N,b", [(2048, 2304, 1793, 256), (2560, 2048, 2047, 512), (2048, 2048, 1992, 128)])
def test_ragged_token_counts_on_the_streaming_kernels(lib, m, n, N, b):
    """Token counts that the layer pads to whole tiles inside the workspace: one past a tile, one short of one, a
    multiple of 8; both layouts, B kept or recomputed (each has its own mix of padded and unpadded tensors), the
    workspace poisoned with NaN so that a stage reading what no stage wrote shows."""
    k = 2
    data = synth_layer(9300 + m + N + b, m, n, N, b, k, "bf16", 0.005)
    ref = orc.linear_fwd_bwd_from_theta(data["X"], data["dZ"], data["W"], data["pi_R"], data["pi_P"],
                                        data["theta_R"], data["theta_P"], b, k)
    check_layer(run_layer(data, "bf16"), ref, data["pi_P"], "bf16")
    bf = torch.bfloat16
    X, dZ, W = (to_dev(data[key], bf) for key in ("X", "dZ", "W"))
    th = {s: to_dev(data["theta_" + s], torch.float32) for s in "RP"}
    pi = {s: torch.from_numpy(data["pi_" + s]).cuda() for s in "RP"}
    blk = {}
    for s, d in (("R", m), ("P", n)):
        blk[s] = torch.empty((th[s].shape[0], 2, b, b), dtype=bf, device="cuda")
        ws = torch.empty(lib.poetx_cnp_workspace_bytes(d, b), dtype=torch.uint8, device="cuda")
        lib.poetx_cnp_build(th[s], d, b, k, lib.CNP_BF16, None, blk[s], ws)
    for layout in (lib.FEATURE_MAJOR, lib.TOKEN_MAJOR):
        tm = layout == lib.TOKEN_MAJOR
        turn = (lambda t: t.t().contiguous()) if tm else (lambda t: t)
        for mem in (False, True):
            desc = lib.make_desc(m, n, b, k, N, lib.BF16, flags=lib.FLAG_RECOMPUTE_B if mem else 0, layout=layout)
            ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
            Z, dX = torch.empty_like(turn(dZ)), torch.empty_like(turn(X))
            B = None if mem else torch.empty((n, N), dtype=bf, device="cuda")
            dth = {s: torch.full_like(th[s], float("nan")) for s in "RP"}
            lib.poetx_linear_fwd(desc, turn(X), W, pi["R"], pi["P"], blk["R"], blk["P"], Z, B, ws)
            lib.poetx_linear_bwd(desc, turn(X), turn(dZ), B, W, pi["R"], pi["P"], blk["R"], blk["P"], th["R"], th["P"], dX,
                                 dth["R"], dth["P"], False, ws)
            torch.cuda.synchronize()
            got = {"Z": to_np(turn(Z)), "dX": to_np(turn(dX)), "dtheta_R": to_np(dth["R"]), "dtheta_P": to_np(dth["P"])}
            for key, v in got.items():
                assert rel_err(v, ref[key]) <= TOL["bf16"], (key, layout, mem)


def layer_calls(lib, data, dtype, layout, mem):
    """Every linear call of one layout on device tensors, activations returned feature major: the forward, the recomputed
    B, the backward in two calls and in one.  mem: B recomputed inside the forward and the one-call backward."""
    m, n, N, b, k = (data[key] for key in ("m", "n", "N", "b", "k"))
    dt, tm = tdtype(dtype), layout == lib.TOKEN_MAJOR
    turn = (lambda t: t.t().contiguous()) if tm else (lambda t: t)
    X, dZ, W = turn(to_dev(data["X"], dt)), turn(to_dev(data["dZ"], dt)), to_dev(data["W"], dt)
    pi = {s: torch.from_numpy(data["pi_" + s].astype(np.int32)).cuda() for s in "RP"}
    th = {s: to_dev(data["theta_" + s], torch.float32) for s in "RP"}
    blk = {s: build_blocks(data["theta_" + s], d, b, k, dtype)[0] for s, d in (("R", m), ("P", n))}
    desc = lib.make_desc(m, n, b, k, N, lib.F32 if dtype == "f32" else lib.BF16, flags=lib.FLAG_RECOMPUTE_B if mem else 0, layout=layout)
    # poisoned: a stage that reads what no stage wrote shows
    ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
    B, dA = (torch.full((d, N), float("nan"), dtype=dt, device="cuda") for d in (n, m))
    Z, dX, dX1 = torch.empty_like(dZ), torch.empty_like(X), torch.empty_like(X)
    two, one = ({s: torch.full_like(th[s], float("nan")) for s in "RP"} for _ in range(2))
    lib.poetx_linear_fwd(desc, X, W, pi["R"], pi["P"], blk["R"], blk["P"], Z, None if mem else B, ws)
    if mem:
        lib.poetx_linear_recompute_b(desc, X, W, pi["R"], blk["R"], B, ws)
    lib.poetx_linear_bwd_input(desc, dZ, W, pi["R"], pi["P"], blk["R"], blk["P"], dX, dA, ws)
    lib.poetx_linear_bwd_skew(desc, X, dZ, B, dA, pi["R"], pi["P"], th["R"], th["P"], two["R"], two["P"], False, ws)
    lib.poetx_linear_bwd(desc, X, dZ, None if mem else B, W, pi["R"], pi["P"], blk["R"], blk["P"], th["R"], th["P"], dX1,
                         one["R"], one["P"], False, ws)
    torch.cuda.synchronize()
    back = (lambda t: t.t().contiguous()) if tm else (lambda t: t)
    return {"Z": back(Z), "B": B, "dX": back(dX), "dA": dA, "one-call dX": back(dX1), "dtheta_R": two["R"], "dtheta_P": two["P"],
            "one-call dtheta_R": one["R"], "one-call dtheta_P": one["P"]}


RAGGED_LAYERS = [
    # unpadded layers: rows of the workspace are rounded up to 8 tokens only
    (1024, 1024, 125, 256, "bf16"),     # 128 columns inside, a whole tile that the caller's tensors do not have
    (1024, 512, 253, 256, "bf16"),      # 256 inside
    (1024, 1024, 61, 512, "bf16"),      # 64 inside
    (512, 768, 255, 64, "bf16"),        # small blocks: the contraction of the block gradients rounds up to a longer one
    (512, 768, 255, 64, "f32"),
    (1024, 768, 250, 192, "bf16"),      # neither small nor a streaming block side
    (2048, 1920, 1660, 64, "f32"),      # 1664 columns inside: multiples of 128, which 1660 tokens are not
    (128, 10240, 1660, 64, "f32"),      # ... and 1040 tiles, enough for the streaming fp32 product, which takes whole tiles of tokens only
    (520, 512, 2045, 8, "bf16"),        # applies of very small blocks on the plain kernel ...
    (520, 512, 2045, 8, "f32"),
    (1056, 768, 2001, 16, "bf16"),      # ... on one side only
    # a handful of tokens
    (512, 768, 1, 256, "bf16"),
    (1024, 512, 7, 512, "bf16"),        # a contraction of four steps per wave, forward, none of the groups of eight
    (2304, 512, 5, 256, "bf16"),        # nine steps per wave: a group and one more
    (1472, 960, 16, 64, "bf16"),
    (256, 384, 17, 128, "bf16"),        # two token tiles
    (768, 512, 32, 256, "bf16"),        # the last that takes the short kernels ...
    (768, 512, 33, 256, "bf16"),
    (2048, 8192, 13, 256, "bf16"),
    (512, 12288, 13, 512, "bf16"),      # four row tiles per workgroup
    (4096, 4608, 17, 512, "bf16"),      # the short kernels refuse this weight from 17 tokens on ...
    (8192, 512, 12, 256, "bf16"),       # ... and for few rows by tokens times contraction: the last that they take
    (8192, 512, 13, 256, "bf16"),
    (4096, 1024, 32, 512, "bf16"),      # ... for more rows
    (4352, 1024, 31, 256, "bf16"),
    # layers that are padded to whole 256-token tiles
    (2048, 2048, 100, 256, "bf16"),     # fewer tokens than a tile
    (2048, 2304, 192, 256, "bf16"),     # a multiple of the 64-token tiles
    (2048, 2560, 200, 512, "bf16"),
    (2048, 2560, 320, 512, "bf16"),
    (4096, 4096, 72, 128, "bf16"),      # small blocks: their tile must not depend on the padding
    (2048, 2048, 1088, 256, "bf16"),    # 17 * 64
    (2048, 2304, 1793, 256, "bf16"),    # one past a tile
]


@pytest.mark.parametrize("m,n,N,b,dtype", RAGGED_LAYERS)
def test_ragged_tokens_give_the_same_activations_in_every_form(lib, m, n, N, b, dtype):
    """Activations (Z, B, dX, dA) of a token count that is no whole tile: bit for bit the same from either layout, from B kept
    or recomputed and from one backward call or two, and right by the oracle."""
    data = synth_layer(9600 + m + n + N + b, m, n, N, b, 2, dtype, 0.01 if b < 256 else 0.005)
    ref = orc.linear_fwd_bwd_from_theta(data["X"], data["dZ"], data["W"], data["pi_R"], data["pi_P"],
                                        data["theta_R"], data["theta_P"], b, 2)
    first = layer_calls(lib, data, dtype, lib.FEATURE_MAJOR, False)
    assert rel_err(to_np(first["Z"]), ref["Z"]) <= TOL[dtype] and rel_err(to_np(first["dX"]), ref["dX"]) <= TOL[dtype]
    assert torch.equal(first["dX"], first["one-call dX"])
    for layout in (lib.FEATURE_MAJOR, lib.TOKEN_MAJOR):
        for mem in (False, True):
            got = layer_calls(lib, data, dtype, layout, mem)
            off = [key for key in ("Z", "B", "dX", "dA", "one-call dX") if not torch.equal(got[key], first[key])]
            assert not off, (off, "token major" if layout else "feature major", "B recomputed" if mem else "B kept")


@pytest.mark.parametrize("m,n,N,b,dtype", RAGGED_LAYERS)
def test_ragged_tokens_give_the_same_parameter_gradients_in_every_form(lib, m, n, N, b, dtype):
    """The packed gradients of the same layers: bit for bit the same from either layout and from B kept or recomputed, in two
    calls and in one (which may differ from each other by the order of a sum), and right by the oracle."""
    data = synth_layer(9600 + m + n + N + b, m, n, N, b, 2, dtype, 0.01 if b < 256 else 0.005)
    ref = orc.linear_fwd_bwd_from_theta(data["X"], data["dZ"], data["W"], data["pi_R"], data["pi_P"],
                                        data["theta_R"], data["theta_P"], b, 2)
    first = layer_calls(lib, data, dtype, lib.FEATURE_MAJOR, False)
    keys = [pre + "dtheta_" + s for s in "RP" for pre in ("", "one-call ")]
    for key in keys:
        assert rel_err(to_np(first[key]), ref[key.split()[-1]]) <= TOL[dtype], key
    for layout in (lib.FEATURE_MAJOR, lib.TOKEN_MAJOR):
        for mem in (False, True):
            got = layer_calls(lib, data, dtype, layout, mem)
            off = [key for key in keys if not torch.equal(got[key], first[key])]
            assert not off, (off, "token major" if layout else "feature major", "B recomputed" if mem else "B kept")


@pytest.mark.parametrize("n,m,N", [
    # tile and contraction ranges that the rule gives the forward; the backward
    (256, 256, 256),        # 128 x 128; the same (contraction too short to split)
    (256, 2048, 256),       # 128 x 128 in 8 ranges; 128 x 128
    (512, 512, 1024),       # 128 x 128; the same
    (2048, 512, 2048),      # 128 x 128; the same
    (2048, 768, 768),       # 128 x 128; 128 x 128 in 4
    (256, 2304, 256),       # 128 x 128 in 8, of ten and eight stages; 128 x 128
    (2304, 256, 256),       # the other way round
    (2304, 2048, 2560),     # 256 x 128, nine tile rows (no whole groups of four); the same with eight
    (4096, 512, 2304),      # 256 x 256, 144 tiles; 128 x 128 in 2
    # ragged counts, padded inside: stores that end at the last token, at rows of odd length
    (2048, 2048, 1801),     # 128 x 128; the same
    (512, 8192, 300),       # 128 x 128 in 8 (ragged reduction); 128 x 128
    (256, 8192, 301),       # 128 x 128 in 16; 128 x 128
    (256, 8704, 301),       # 128 x 128 in 16, of 18 and 16 stages; 256 x 128
    (512, 2048, 1001),      # 128 x 128 in 4; 128 x 128
    (768, 2560, 1501),      # 128 x 128 in 2; 128 x 128
    (4096, 512, 1100),      # 256 x 128; 128 x 128 in 4
    (2304, 2048, 2559),     # 256 x 128; the same
    (4096, 512, 2300),      # 256 x 256; 128 x 128 in 2
    (512, 2560, 3329),      # 128 x 128; 256 x 256
])
def test_dense_tiles(lib, n, m, N):
    """Every output tile of the streaming bf16 product, whole and ragged, and split contractions, both directions, against float64 on the same
    bf16 operands: a whole pass with blocks equal to the identity is the dense product between two exact
    permutation round trips.  One bf16 rounding of an fp32 sum: 2^-8 of the largest value is generous."""
    rng = np.random.Generator(np.random.PCG64(9400 + n + m + N))
    b = 256
    X, dZ = round_bf16(rng.standard_normal((m, N))), round_bf16(rng.standard_normal((n, N)))
    W = round_bf16(rng.standard_normal((n, m)) * 0.02)
    bf = torch.bfloat16
    desc = lib.make_desc(m, n, b, 2, N, lib.BF16)
    ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
    pi = {"R": torch.from_numpy(rng.permutation(m).astype(np.int32)).cuda(), "P": torch.from_numpy(rng.permutation(n).astype(np.int32)).cuda()}
    blk = {s: torch.zeros((d // b, 2, b, b), dtype=bf, device="cuda") for s, d in (("R", m), ("P", n))}
    Xd, dZd, Wd = to_dev(X, bf), to_dev(dZ, bf), to_dev(W, bf)
    guard, guard_dA = (torch.full((d * N + 512,), -7.0, dtype=bf, device="cuda") for d in (n, m))
    Z, B = torch.empty((n, N), dtype=bf, device="cuda"), guard[256:256 + n * N].view(n, N)
    dX, dA = torch.empty((m, N), dtype=bf, device="cuda"), guard_dA[256:256 + m * N].view(m, N)
    lib.poetx_linear_fwd(desc, Xd, Wd, pi["R"], pi["P"], blk["R"], blk["P"], Z, B, ws)
    lib.poetx_linear_bwd_input(desc, dZd, Wd, pi["R"], pi["P"], blk["R"], blk["P"], dX, dA, ws)
    torch.cuda.synchronize()
    assert rel_err(to_np(B), W @ X) <= 2.0 ** -8 and torch.equal(Z, B)
    assert rel_err(to_np(dA), W.T @ dZ) <= 2.0 ** -8 and torch.equal(dX, dA)
    for buf, used in ((guard, n * N), (guard_dA, m * N)):
        assert torch.all(buf[:256] == -7.0) and torch.all(buf[256 + used:] == -7.0)


@pytest.mark.parametrize("dtype,n,m,N", [
    # tile and contraction ranges of the sliced product, forward; backward
    ("f32", 64, 48, 5),          # 32 x 32, fewer slices than waves; the same
    ("f32", 256, 256, 512),      # 32 x 32; the same
    ("f32", 1024, 768, 1001),    # 64 x 64, columns over; 32 x 32
    ("f32", 1040, 1008, 1991),   # 32 x 32, half a tile of rows over; 64 x 64, rows and columns over
    ("f32", 432, 1840, 583),     # 64 x 64 in ranges, a quarter tile of rows over; 32 x 64
    ("f32", 1808, 336, 759),     # 32 x 64, rows and columns over; 64 x 64 in ranges
    ("f32", 3440, 304, 271),     # 32 x 32; 32 x 64 in ranges
    ("f32", 144, 3264, 33),      # 32 x 32 in ranges; 32 x 32
    ("f32", 1792, 16, 40),       # one slice: seven waves without any; 32 x 32 in ranges
    ("f32", 4112, 4096, 2040),   # 64 x 64, large weight
    ("bf16", 64, 96, 3),         # 32 x 32, three slices for eight waves; two
    ("bf16", 512, 1376, 1024),   # 32 x 64; the same
    ("bf16", 1376, 512, 1023),   # 32 x 64; the same
    ("bf16", 96, 3200, 17),      # 32 x 32 in ranges; 32 x 32
    ("bf16", 2208, 32, 43),      # 32 x 32; 32 x 64 in ranges
    ("bf16", 32, 1984, 40),      # the other way round
    ("bf16", 432, 3104, 270),    # 64 x 64 in ranges; not in slices (432 are none)
    ("bf16", 3968, 784, 207),    # the other way round
    ("bf16", 3104, 2080, 29),    # few columns of a large weight: 32 x 32; 64 x 32 in ranges
    ("bf16", 1344, 2400, 7),     # 32 x 32 in ranges; 64 x 32 in ranges
    ("bf16", 1056, 3072, 16),    # 32 x 32 in ranges; 64 x 32
    ("bf16", 2080, 3104, 300),   # large weight: 64 x 64 by price; the same
    ("bf16", 3584, 2464, 295),   # edge tiles by price; 64 x 64
    ("bf16", 1568, 1504, 2999),  # 64 x 64; the same
    ("f32", 4128, 96, 2056),     # many tiles of a short contraction: the edge kernel; 32 x 32
    ("f32", 4128, 176, 2056),    # not short: 64 x 64; 64 x 64 in ranges
    ("bf16", 3104, 64, 2999),    # the edge kernel; 32 x 32
    ("bf16", 64, 3104, 2999),    # ... in the backward
    ("bf16", 1568, 64, 1999),    # 208 tiles of 128 x 128 of a short contraction: the edge kernel; 32 x 32
    ("bf16", 64, 1568, 1999),    # ... in the backward
    ("bf16", 64, 3104, 1601),    # 325 of them in the backward: slices
    ("bf16", 4128, 128, 1201),   # 330: the edge kernel by price
])
def test_sliced_dense_products(lib, dtype, n, m, N):
    """The sliced product at the edges of its tiles, with fewer slices than waves and with split contractions, both directions, against float64 on the same operands, nothing written outside; and
    against the general kernel, which the same call takes when the weight lies one element off a 16-byte boundary.  A whole pass with blocks equal to the
    identity is the dense product between two exact permutation round trips.  fp32: K additions rounded by 2^-24 of a running sum no larger than the
    largest result, which add up like a random walk: sqrt(4112) 2^-24 = 3.8e-6; bf16: one rounding more, 2^-9."""
    rng = np.random.Generator(np.random.PCG64(9900 + n + m + N))
    b, dt, tol = 16, tdtype(dtype), (4e-6 if dtype == "f32" else 2.0 ** -8)
    rnd = round_f32 if dtype == "f32" else round_bf16
    X, dZ = rnd(rng.standard_normal((m, N))), rnd(rng.standard_normal((n, N)))
    W = rnd(rng.standard_normal((n, m)) * 0.02)
    desc = lib.make_desc(m, n, b, 2, N, lib.F32 if dtype == "f32" else lib.BF16)
    pi = {"R": torch.from_numpy(rng.permutation(m).astype(np.int32)).cuda(), "P": torch.from_numpy(rng.permutation(n).astype(np.int32)).cuda()}
    if dtype == "f32":
        blk = {s: torch.eye(b, device="cuda").repeat(d // b, 1, 1).contiguous() for s, d in (("R", m), ("P", n))}
    else:
        blk = {s: torch.zeros((d // b, 2, b, b), dtype=dt, device="cuda") for s, d in (("R", m), ("P", n))}
    Xd, dZd = to_dev(X, dt), to_dev(dZ, dt)
    got = []
    for off in (0, 1):
        Wd = torch.empty(n * m + 1, dtype=dt, device="cuda")[off:off + n * m].view(n, m)
        Wd.copy_(to_dev(W, dt))
        ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
        guard, guard_dA = (torch.full((d * N + 512,), -7.0, dtype=dt, device="cuda") for d in (n, m))
        Z, B = torch.empty((n, N), dtype=dt, device="cuda"), guard[256:256 + n * N].view(n, N)
        dX, dA = torch.empty((m, N), dtype=dt, device="cuda"), guard_dA[256:256 + m * N].view(m, N)
        lib.poetx_linear_fwd(desc, Xd, Wd, pi["R"], pi["P"], blk["R"], blk["P"], Z, B, ws)
        lib.poetx_linear_bwd_input(desc, dZd, Wd, pi["R"], pi["P"], blk["R"], blk["P"], dX, dA, ws)
        torch.cuda.synchronize()
        assert rel_err(to_np(B), W @ X) <= tol and torch.equal(Z, B)
        assert rel_err(to_np(dA), W.T @ dZ) <= tol and torch.equal(dX, dA)
        for buf, used in ((guard, n * N), (guard_dA, m * N)):
            assert torch.all(buf[:256] == -7.0) and torch.all(buf[256 + used:] == -7.0)
        got.append((to_np(B), to_np(dA)))
    for here, general in zip(*got):
        assert rel_err(here, general) <= tol


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,n,N,b", [
    (256, 256, 512, 32),      # whole tiles throughout, apply on 32 x 32
    (512, 1376, 1024, 64),    # a ragged last block on one side only
    (768, 1024, 1001, 64),    # apply on 64 x 64, tails
    (384, 256, 30, 128),      # stages of half a block, fewer tokens than a tile
    (130, 75, 5, 65),         # last blocks of one row and of ten, rows shorter than a vector
    (2048, 64, 4096, 64),     # 64 x 64 gradients: two launches
])
def test_apply_and_block_gradients_in_one_launch(lib, m, n, N, b, dtype):
    """The one-call backward of small blocks launches dX = R dA and both block gradients together where their tiles allow it: the same tiles, so the same bits as the two halves."""
    rng = np.random.Generator(np.random.PCG64(9950 + m + n + N + b))
    dt, k = tdtype(dtype), 3
    code = lib.F32 if dtype == "f32" else lib.BF16
    t = lambda *shape: torch.from_numpy(rng.standard_normal(shape)).to("cuda", dt)
    X, dZ, B, W = t(m, N), t(n, N), t(n, N), t(n, m) * 0.02
    nR, nP = -(-m // b), -(-n // b)
    pi = [torch.from_numpy(rng.permutation(d).astype(np.int32)).cuda() for d in (m, n)]
    blk = [t(nb, b, b) * 0.1 if dtype == "f32" else t(nb, 2, b, b) * 0.1 for nb in (nR, nP)]
    th = [torch.from_numpy(rng.standard_normal((nb, b * (b - 1) // 2)) * 0.01).to("cuda", torch.float32) for nb in (nR, nP)]
    desc = lib.make_desc(m, n, b, k, N, code)
    got = []
    for one in (True, False):
        ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
        dX, dA = torch.full_like(X, float("nan")), torch.empty_like(X)
        dth = [torch.full_like(x, float("nan")) for x in th]
        if one:
            lib.poetx_linear_bwd(desc, X, dZ, B, W, *pi, *blk, *th, dX, *dth, False, ws)
        else:
            lib.poetx_linear_bwd_input(desc, dZ, W, *pi, *blk, dX, dA, ws)
            lib.poetx_linear_bwd_skew(desc, X, dZ, B, dA, *pi, *th, *dth, False, ws)
        torch.cuda.synchronize()
        got.append((dX, *dth))
    for one, two in zip(*got):
        assert torch.all(torch.isfinite(one)) and torch.equal(one, two)


@pytest.mark.parametrize("m,n,N", [
    (5376, 256, 7936),    # 21 blocks of 124 tiles over 128 pairs: shares of 20 and 21, borders anywhere in a share
    (256, 33280, 1280),   # 130 blocks of 20 tiles: blocks that one pair covers whole, and a border at nearly every share
    (2816, 2816, 16384),  # both sides, 11 blocks of 256 tiles: 22 a share
])
def test_block_stage_over_block_borders(lib, m, n, N):
    """One-pass backward whose workgroups take equal shares of all blocks' tiles: the two halves' bits for dX, and every block gradient as its own sum in fp64."""
    g = torch.Generator(device="cuda").manual_seed(9980 + m + n + N)
    r = lambda *shape: torch.randn(*shape, device="cuda", dtype=torch.float32, generator=g).to(torch.bfloat16)
    b = 256
    X, dZ, B, W = r(m, N), r(n, N), r(n, N), r(n, m) * 0.02
    pi = [torch.randperm(d, device="cuda", generator=g).to(torch.int32) for d in (m, n)]
    blk = [r(d // b, 2, b, b) * 0.01 for d in (m, n)]
    th = [torch.zeros(d // b, b * (b - 1) // 2, device="cuda") for d in (m, n)]
    desc = lib.make_desc(m, n, b, 3, N, lib.BF16, flags=lib.FLAG_BLOCK_GRADS)
    assert lib.poetx_linear_path(desc) & lib.PATH_BWD_ONE_PASS
    ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
    dX, dX2, dA = torch.full_like(X, float("nan")), torch.full_like(X, float("nan")), torch.empty_like(X)
    dG = [torch.full((d // b, b, b), float("nan"), device="cuda") for d in (m, n)]
    lib.poetx_linear_bwd(desc, X, dZ, B, W, *pi, *blk, *th, dX, *dG, False, ws)
    lib.poetx_linear_bwd_input(desc, dZ, W, *pi, *blk, dX2, dA, ws)
    torch.cuda.synchronize()
    assert torch.equal(dX, dX2)
    for U, V, p, got in ((X, dA, pi[0], dG[0]), (B, dZ, pi[1], dG[1])):
        p = p.long()
        for j in range(got.shape[0]):
            rows = p[j * b:(j + 1) * b]
            ref = U[rows].double() @ V[rows].double().t()
            # a sum of N products in fp32, each addition off by 2^-24 of what it adds to; they add up like a walk, at most by their number's root times 4
            assert (got[j].double() - ref).abs().max() <= 4 * N ** 0.5 * 2.0 ** -24 * ref.abs().max()


@pytest.mark.parametrize("m,n,N,b", [
    (1024, 768, 65600, 256),   # 1025 * 64 tokens: one range, on 768 features just beyond the line of 2^25 elements
    (512, 768, 65664, 256),    # 1026 * 64: two ranges of an odd number of stages
    (512, 1024, 65664, 512),   # four tiles of a block
    (5376, 512, 66560, 512),   # 1040 * 64, 512 features: sixteen ranges of 65; 5376 = 10.5 * 512: the other side on the edge kernel
])
def test_streaming_block_gradients(lib, m, n, N, b):
    """Block gradients of long streams, two-call backward, on the kernel of whole 64-token stages: both layouts (rows as long as the tokens, and padded ones) the same bits, and every
    block as its own sum in fp64."""
    g = torch.Generator(device="cuda").manual_seed(9990 + m + n + N)
    r = lambda *shape: torch.randn(*shape, device="cuda", dtype=torch.float32, generator=g).to(torch.bfloat16)
    X, dZ, B, dA = r(m, N), r(n, N), r(n, N), r(m, N)
    pi = [torch.randperm(d, device="cuda", generator=g).to(torch.int32) for d in (m, n)]
    nb = [-(-d // b) for d in (m, n)]
    th = [torch.zeros(k, b * (b - 1) // 2, device="cuda") for k in nb]
    first = None
    for layout in (lib.FEATURE_MAJOR, lib.TOKEN_MAJOR):
        desc = lib.make_desc(m, n, b, 2, N, lib.BF16, flags=lib.FLAG_BLOCK_GRADS, layout=layout)
        assert m % b or lib.poetx_linear_path(desc) & lib.PATH_BLOCKGRAD
        ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
        turn = (lambda t: t.t().contiguous()) if layout == lib.TOKEN_MAJOR else (lambda t: t)
        dG = [torch.full((k, b, b), float("nan"), device="cuda") for k in nb]
        lib.poetx_linear_bwd_skew(desc, turn(X), turn(dZ), B, dA, *pi, *th, *dG, False, ws)
        torch.cuda.synchronize()
        first = first or dG
        assert all(torch.equal(a, c) for a, c in zip(dG, first))
    for U, V, p, got in ((X, dA, pi[0], dG[0]), (B, dZ, pi[1], dG[1])):
        p = p.long()
        for j in range(got.shape[0]):
            rows = p[j * b:(j + 1) * b]
            ref = torch.zeros((b, b), dtype=torch.float64, device="cuda")
            ref[:rows.numel(), :rows.numel()] = U[rows].double() @ V[rows].double().t()
            # a sum of N products in fp32, each addition off by 2^-24 of what it adds to; they add up like a walk, at most by their number's root times 4
            assert (got[j].double() - ref).abs().max() <= 4 * N ** 0.5 * 2.0 ** -24 * ref.abs().max()


@pytest.mark.parametrize("b,nb,ks", [(512, 2, (1, 2, 3, 4, 5, 6)), (512, 40, (3,)), (512, 130, (3,)), (256, 130, (2,)), (256, 150, (2,)), (256, 3, (1, 2, 7)), (256, 9, (1, 5)), (256, 200, (4,))])
def test_matrix_core_series(lib, b, nb, ks):
    """The bf16 series of large blocks, build and backward through poetx_cnp_build / poetx_cnp_bwd: every shape of the
    recurrences (the tiled one pairs powers: odd and even orders start differently), batches that the tiled one of b = 512 works off
    in more than one group and that fill the chip once, in part and more than once in the one launch of b = 256.  The bound is the error of rounding each product's operands
    to bf16 (2^-9 of the first product, relative to terms of its size) with a factor of four."""
    L = b * (b - 1) // 2
    for k in ks:
        rng = np.random.Generator(np.random.PCG64(9500 + b + nb + k))
        theta = round_f32(rng.standard_normal((nb, L)) * 0.008)
        check = sorted({0, nb // 2, nb - 1})
        th = to_dev(theta, torch.float32)
        G = torch.empty((nb, b, b), dtype=torch.float32, device="cuda")
        E = torch.empty((nb, 2, b, b), dtype=torch.bfloat16, device="cuda")
        d = nb * b
        ws = torch.full((max(lib.poetx_cnp_workspace_bytes(d, b), lib.poetx_cnp_bwd_workspace_bytes(d, b, k)) // 4,), float("nan"),
                        dtype=torch.float32, device="cuda").view(torch.uint8)
        lib.poetx_cnp_build(th, d, b, k, lib.CNP_BF16, G, E, ws)
        dG = torch.randn((nb, b, b), generator=torch.Generator(device="cuda").manual_seed(k), device="cuda")
        dth = torch.full_like(th, float("nan"))
        lib.poetx_cnp_bwd(th, dG, d, b, k, lib.CNP_BF16, dth, False, ws)
        torch.cuda.synchronize()
        Q = orc.skew_from_packed(theta[check], b, len(check) * b)
        ref = orc.cnp(Q, k) - np.eye(b)
        norm = np.linalg.norm(Q[0], 2)
        assert np.linalg.norm(to_np(G)[check] - np.eye(b) - ref) <= 4 * 2.0 ** -9 * norm * np.linalg.norm(ref)
        assert np.linalg.norm(to_np(E[check])[:, 0] - ref) <= (2.0 ** -8 + 4 * 2.0 ** -9 * norm) * np.linalg.norm(ref)
        assert torch.equal(E[:, 1], E[:, 0].transpose(1, 2))
        want = orc.packed_from_skew_grad(orc.cnp_bwd(Q, to_np(dG)[check], k), b, len(check) * b)
        assert np.linalg.norm(to_np(dth)[check] - want) <= 4 * 2.0 ** -9 * norm * np.linalg.norm(want)


def test_column_counts_up_to_the_last_int(lib):
    """2^31 - 5 tokens of two features: column indices run up to the last int, and the tiles need more workgroups than one grid
    dimension holds.  Tokens are zero but for runs at the ends and where an index or a grid could wrap; the apply, the
    forward and the block gradients against float64 there, and finite (written, from zeros) everywhere else."""
    m, N, b, bf = 2, 2 ** 31 - 5, 2, torch.bfloat16
    at = torch.cat([torch.arange(max(c - 40, 0), min(c + 40, N)) for c in (0, 2 ** 24, 2 ** 29, 2 ** 30, N)]).cuda()
    g = torch.Generator(device="cuda").manual_seed(1)

    def sparse():
        t = torch.zeros((m, N), dtype=bf, device="cuda")
        t[:, at] = torch.randn((m, at.numel()), generator=g, device="cuda").to(bf)
        return t, t[:, at].double()
    X, x = sparse()
    E = (torch.randn((1, b, b), generator=g, device="cuda") * 0.1).to(bf)
    blk, G = torch.stack((E, E.transpose(1, 2)), 1).contiguous(), E[0].double() + torch.eye(b, device="cuda", dtype=torch.float64)
    W = torch.randn((m, m), generator=g, device="cuda").to(bf)
    pi = torch.tensor([1, 0], dtype=torch.int32, device="cuda")
    swap = lambda t: t.flip(0)
    err = lambda got, want: float((got[:, at].double() - want).norm() / want.norm())
    Z = torch.full_like(X, float("nan"))
    lib.poetx_perm_blockdiag_apply_left(X, Z, pi, blk, b, False)
    torch.cuda.synchronize()
    assert err(Z, swap(G @ swap(x))) <= 2.0 ** -8 and bool(torch.isfinite(Z).all())
    desc = lib.make_desc(m, m, b, 1, N, lib.BF16, flags=lib.FLAG_BLOCK_GRADS)
    ws = torch.empty(lib.poetx_linear_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    B = torch.full_like(X, float("nan"))
    Z.fill_(float("nan"))
    lib.poetx_linear_fwd(desc, X, W, pi, pi, blk, blk, Z, B, ws)
    torch.cuda.synchronize()
    want = W.double() @ swap(G.T @ swap(x))
    assert err(B, want) <= 2.0 ** -7 and bool(torch.isfinite(B).all())
    assert err(Z, swap(G.T @ swap(want))) <= 2.0 ** -6 and bool(torch.isfinite(Z).all())
    del Z
    dZ, z = sparse()
    th = torch.zeros((1, 1), device="cuda")
    dG = {s: torch.full((1, b, b), float("nan"), device="cuda") for s in "RP"}
    lib.poetx_linear_bwd_skew(desc, X, dZ, B, dZ, pi, pi, th, th, dG["R"], dG["P"], False, ws)   # dZ in dA's place
    torch.cuda.synchronize()
    for s, u in (("R", x), ("P", B[:, at].double())):
        want = swap(u) @ swap(z).T
        assert float((dG[s][0].double() - want).norm() / want.norm()) <= 1e-5, s


def test_block_counts_beyond_one_grid_dimension(lib):
    """35 million 2 x 2 blocks: build, backward and apply need more workgroups than a grid dimension holds.  A block is
    [[0, t], [-t, 0]], so at k = 2 the series is (1 - 2 t^2) I + (2 t - t^3) J."""
    d, b, k = 70_000_001, 2, 2
    nb = (d + 1) // 2
    g = torch.Generator(device="cuda").manual_seed(2)
    th = torch.randn((nb, 1), generator=g, device="cuda") * 0.1
    live = th[:, 0].clone()
    live[-1] = 0.0                                   # a tail block of side one: its parameter is dead
    ws = torch.empty(max(lib.poetx_cnp_workspace_bytes(d, b), lib.poetx_cnp_bwd_workspace_bytes(d, b, k)), dtype=torch.uint8, device="cuda")
    G = torch.full((nb, b, b), float("nan"), device="cuda")
    lib.poetx_cnp_build(th, d, b, k, lib.CNP_FP32, G, None, ws)
    diag, off = 1 - 2 * live ** 2, 2 * live - live ** 3
    want = torch.stack((diag, off, -off, diag), 1).view(nb, b, b)
    assert float((G - want).abs().max()) <= 1e-6
    dG = torch.randn((nb, b, b), generator=g, device="cuda")
    dth = torch.full_like(th, float("nan"))
    lib.poetx_cnp_bwd(th, dG, d, b, k, lib.CNP_FP32, dth, False, ws)
    grad = -4 * live * (dG[:, 0, 0] + dG[:, 1, 1]) + (2 - 3 * live ** 2) * (dG[:, 0, 1] - dG[:, 1, 0])
    grad[-1] = 0.0
    assert float((dth[:, 0] - grad).abs().max()) <= 1e-5
    pi = torch.randperm(d, generator=g, device="cuda")
    V = torch.randn((d, 1), generator=g, device="cuda")
    out = torch.full_like(V, float("nan"))
    lib.poetx_perm_blockdiag_apply_left(V, out, pi.to(torch.int32), G, b, False)
    x = torch.zeros(nb * b, device="cuda")
    x[:d] = V[pi, 0]
    y = (G * x.view(nb, 1, b)).sum(2).view(-1)[:d]
    assert float((out[pi, 0] - y).abs().max()) <= 1e-5


def test_contraction_of_two_to_the_29(lib):
    """A backward product over 2^29 output features, fp32: its operand's row of 2^31 bytes is past what an int counts.  Blocks of one, equal to one, and the identity
    order, so that dA = W^T dZ; features are zero but for runs at the ends and where a count or an offset could wrap."""
    m, n, b = 4, 2 ** 29, 1
    g = torch.Generator(device="cuda").manual_seed(3)
    at = torch.cat([torch.arange(max(c - 20, 0), min(c + 20, n)) for c in (0, 2 ** 25, 2 ** 27, 2 ** 28, n)]).cuda()
    W, dZ = torch.zeros((n, m), device="cuda"), torch.zeros((n, 1), device="cuda")
    W[at] = torch.randn((at.numel(), m), generator=g, device="cuda")
    dZ[at] = torch.randn((at.numel(), 1), generator=g, device="cuda")
    pi = torch.arange(n, dtype=torch.int32, device="cuda")
    one = torch.ones((n, 1, 1), device="cuda")
    desc = lib.make_desc(m, n, b, 1, 1, lib.F32)
    ws = torch.empty(lib.poetx_linear_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    dX, dA = (torch.full((m, 1), float("nan"), device="cuda") for _ in range(2))
    lib.poetx_linear_bwd_input(desc, dZ, W, pi[:m], pi, one[:m], one, dX, dA, ws)
    torch.cuda.synchronize()
    want = W[at].double().T @ dZ[at].double()
    assert float((dA.double() - want).norm() / want.norm()) <= 1e-6 and torch.equal(dX, dA)


def test_one_call_backward_of_blocks_beyond_one_grid_dimension(lib):
    """The whole backward of one token where one side has a single 2 x 2 block and the other 35 million: more gradient workgroups than a grid dimension
    holds, beside an apply of one.  Series gradient of a 2 x 2 block at k = 2 as in the test above."""
    m, n, b, k = 2, 70_000_000, 2, 2
    g = torch.Generator(device="cuda").manual_seed(4)
    r = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    th = {"R": r(1, 1) * 0.1, "P": r(n // b, 1) * 0.1}
    pi = {"R": torch.tensor([1, 0], device="cuda"), "P": torch.randperm(n, generator=g, device="cuda")}

    def block(t):
        t = t[:, 0]
        diag, off = 1 - 2 * t ** 2, 2 * t - t ** 3
        return torch.stack((diag, off, -off, diag), 1).view(-1, b, b).contiguous()
    blk = {s: block(th[s]) for s in "RP"}
    X, dZ, B, W = r(m, 1), r(n, 1), r(n, 1), r(n, m) * 0.02
    desc = lib.make_desc(m, n, b, k, 1, lib.F32)
    ws = torch.empty(lib.poetx_linear_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    dX, dth = torch.full_like(X, float("nan")), {s: torch.full_like(th[s], float("nan")) for s in "RP"}
    p32 = {s: pi[s].to(torch.int32) for s in "RP"}
    lib.poetx_linear_bwd(desc, X, dZ, B, W, p32["R"], p32["P"], blk["R"], blk["P"], th["R"], th["P"], dX, dth["R"], dth["P"], False, ws)
    torch.cuda.synchronize()

    def apply(v, s):
        out = torch.empty_like(v)
        out[pi[s], 0] = (blk[s].double() * v[pi[s], 0].view(-1, 1, b)).sum(2).view(-1)
        return out

    def series_grad(u, v, s):
        d, t = u[pi[s], 0].view(-1, b, 1) * v[pi[s], 0].view(-1, 1, b), th[s][:, 0].double()
        return -4 * t * (d[:, 0, 0] + d[:, 1, 1]) + (2 - 3 * t ** 2) * (d[:, 0, 1] - d[:, 1, 0])
    dA = W.double().T @ apply(dZ.double(), "P")
    err = lambda got, want: float((got.double() - want).norm() / want.norm())
    assert err(dX, apply(dA, "R")) <= 1e-5
    assert err(dth["P"][:, 0], series_grad(B.double(), dZ.double(), "P")) <= 1e-6
    assert err(dth["R"][:, 0], series_grad(X.double(), dA, "R")) <= 1e-5


@pytest.mark.parametrize("b,nbR,nbP", [
    (512, 60, 30),      # groups 64 + 26: the P side ends inside the first group, the R side goes on in the second
    (512, 16, 70),      # the P side ends inside the second group
    (512, 20, 64),      # exactly at the boundary
    (256, 100, 60),     # the sides' boundary early in the one launch over all blocks
    (256, 20, 140),     # late in it
])
def test_series_groups_of_two_sides(lib, b, nbR, nbP):
    """The series backward of both sides of a layer in one batch (several groups of blocks of 512, one launch for those of 256): packed
    gradients bit for bit those of poetx_cnp_bwd, side by side, on the block gradients that the same layer reports."""
    m, n, N, k, bf = nbR * b, nbP * b, 64, 3, torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(b + nbR)
    normal = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    X, dZ, B, dA = (normal(d, N).to(bf) for d in (m, n, n, m))
    pi = {s: torch.randperm(d, generator=g, device="cuda").to(torch.int32) for s, d in (("R", m), ("P", n))}
    th = {s: normal(nb, b * (b - 1) // 2) * 0.005 for s, nb in (("R", nbR), ("P", nbP))}

    def skew(flags, out):
        desc = lib.make_desc(m, n, b, k, N, lib.BF16, flags=flags)
        ws = torch.full((lib.poetx_linear_workspace_bytes(desc) // 4,), float("nan"), dtype=torch.float32, device="cuda").view(torch.uint8)
        lib.poetx_linear_bwd_skew(desc, X, dZ, B, dA, pi["R"], pi["P"], th["R"], th["P"], out["R"], out["P"], False, ws)
        return out
    got = skew(0, {s: torch.full_like(th[s], float("nan")) for s in "RP"})
    dG = skew(lib.FLAG_BLOCK_GRADS, {s: torch.full((nb, b, b), float("nan"), device="cuda") for s, nb in (("R", nbR), ("P", nbP))})
    for s, d in (("R", m), ("P", n)):
        want = torch.full_like(th[s], float("nan"))
        ws = torch.empty(lib.poetx_cnp_bwd_workspace_bytes(d, b, k), dtype=torch.uint8, device="cuda")
        lib.poetx_cnp_bwd(th[s], dG[s], d, b, k, lib.CNP_BF16, want, False, ws)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(want).all()) and torch.equal(got[s], want), s
