"""GPU parity at the edges of the kernels' dispatch: the smallest and largest
size of a variant, and sizes just off its tiles.  Same oracle, metric and
tolerances as test_gpu_parity.py."""
import pytest

from _gpu_helpers import announce
from test_gpu_parity import check_layer, layer_case, oracle_layer, run_layer_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def run_case(T, B, I, H, Hp, dtype, reverse, scale, states=True):
    label = f"edge T{T} B{B} I{I} H{H} Hp{Hp} {dtype} rev{int(reverse)} states{int(states)}"
    announce(label)
    c = layer_case(T, B, I, H, Hp, dtype, reverse, seed=T * 1000 + B + H, states=states, final_grads=states,
                   scale=scale)
    gpu = run_layer_gpu(c, T, B, I, H, Hp, dtype, reverse)
    check_layer(gpu, oracle_layer(c, Hp, reverse), dtype, label)
    return gpu


# XCD-local kernels at widths padded to the next of 256, 512 and 1024:
# (T, B, H, reverse, states); weights U(+-1/sqrt(H)), the usual LSTM range
XCD_PAD_CASES = [
    (3, 5, 8, False, True),       # one workgroup per XCD, one wave's worth of k
    (3, 130, 248, True, True),    # one row of cells short of 256; two row blocks
    (2, 264, 120, False, False),  # four row blocks
    (4, 9, 264, False, True),     # just past 256
    (3, 140, 504, True, False),
    (3, 40, 520, True, True),     # just past 512: half of the workgroups idle
    (4, 130, 648, False, True),   # the last workgroup with a quarter of its cells
    (2, 257, 1016, True, True),   # one workgroup short of full; four row blocks
    (1, 1, 776, False, True),
]


@pytest.mark.parametrize("T,B,H,reverse,states", XCD_PAD_CASES)
def test_padded_xcd_widths(T, B, H, reverse, states):
    gpu = run_case(T, B, 40, H, 0, "bf16", reverse, H ** -0.5, states)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert gpu["tiling"][3] == 1001 and gpu["tiling"][7] == 1001, gpu["tiling"]


# Pipelined row blocks of the XCD-local kernels (33 to 64 rows per XCD, three
# or four blocks, the last XCD and the last block ragged), at every width's
# kernel: (T, B, H, reverse, states)
XCD_BLOCK_CASES = [
    (4, 257, 256, False, True),    # 33 rows per XCD: a third block of one row; the last XCD 26 rows
    (3, 384, 512, True, True),     # three whole blocks
    (2, 505, 1024, False, False),  # four blocks, the last XCD one row short
    (1, 300, 256, False, True),    # one step: nothing to exchange but dh0
    (1, 300, 256, True, False),
    (3, 390, 360, False, True),    # padded width, four blocks
]


@pytest.mark.parametrize("T,B,H,reverse,states", XCD_BLOCK_CASES)
def test_pipelined_row_blocks(T, B, H, reverse, states):
    gpu = run_case(T, B, 40, H, 0, "bf16", reverse, H ** -0.5, states)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert gpu["tiling"][3] in (1000, 1001), gpu["tiling"]


# Generic persistent kernels (fp32, LSTMP, bf16 wider than 1024): (T, B, I, H,
# Hp, dtype, reverse, states).  Between them tiles of 16 and 32 rows, weights in
# LDS and streamed, projections with fewer and with more column blocks than
# workgroups; several tiles per workgroup and tiles of 64 rows are below.
GENERIC_CASES = [
    (3, 1, 8, 8, 0, "f32", False, True),
    (4, 16, 24, 256, 0, "f32", True, True),       # whole tiles
    (3, 33, 24, 264, 0, "f32", False, False),     # one row past two row blocks, half a chunk of k
    (2, 150, 16, 72, 0, "f32", True, True),       # ten row blocks
    (2, 530, 16, 136, 0, "f32", False, True),     # several tiles per workgroup: carries through memory
    (3, 20, 16, 1024, 0, "f32", False, True),     # full-width fp32
    (2, 18, 16, 1160, 0, "f32", True, True),      # weights of a backward slice beyond LDS: streamed
    (3, 17, 16, 1032, 0, "bf16", False, True),    # bf16 just past the XCD-local widths
    (2, 70, 16, 1544, 0, "bf16", True, True),
    (3, 6, 16, 40, 8, "f32", False, True),        # LSTMP: half a column block
    (3, 40, 24, 16, 200, "bf16", True, True),     # more column blocks than workgroups
    (3, 65, 24, 520, 136, "bf16", False, False),
    (2, 19, 24, 1800, 256, "bf16", False, True),
    (2, 36, 24, 640, 320, "f32", True, True),
    (3, 300, 24, 64, 32, "bf16", False, True),    # ten tiles of 32 rows, eight shares of the projection
]


@pytest.mark.parametrize("T,B,I,H,Hp,dtype,reverse,states", GENERIC_CASES)
def test_generic_kernels(T, B, I, H, Hp, dtype, reverse, states):
    gpu = run_case(T, B, I, H, Hp, dtype, reverse, min(0.3, H ** -0.5), states)
    assert gpu["tiling"][3] not in (1000, 1001, 2000), gpu["tiling"]


# Generic tilings with several tiles per workgroup (carries through memory, a
# projection's share striding over the group's tiles) or 64-row tiles, and bf16
# plain layers of more than 512 rows: the case as above, then per direction
# (rows per tile, tiles per workgroup, slice in LDS, projection in LDS)
GENERIC_TILINGS = [
    ((3, 96, 24, 1024, 512, "bf16", False, True), (16, 2, 1, 1), (16, 2, 1, 1)),
    ((2, 128, 24, 1504, 512, "bf16", True, True), (16, 4, 1, 1), (32, 4, 1, 0)),
    ((2, 96, 16, 1024, 512, "f32", False, True), (16, 3, 1, 1), (16, 2, 1, 0)),
    ((2, 64, 16, 1800, 768, "f32", True, False), (16, 2, 0, 1), (16, 2, 1, 0)),   # a streamed slice of R
    ((3, 600, 24, 200, 64, "f32", True, True), (32, 2, 1, 1), (16, 3, 1, 1)),
    ((3, 1100, 16, 40, 24, "bf16", False, True), (64, 2, 1, 1), (64, 2, 1, 1)),
    ((2, 600, 16, 72, 0, "bf16", False, True), (64, 1, 1, 0), (64, 1, 1, 0)),
    ((3, 1100, 16, 40, 0, "bf16", True, True), (64, 2, 1, 0), (64, 2, 1, 0)),
    ((3, 700, 16, 16, 0, "f32", False, True), (64, 1, 1, 0), (64, 1, 1, 0)),
    ((2, 530, 16, 1024, 0, "bf16", False, False), (32, 9, 1, 0), (16, 9, 1, 0)),
]


@pytest.mark.parametrize("case,fwd,bwd", GENERIC_TILINGS)
def test_generic_tilings(case, fwd, bwd):
    T, B, I, H, Hp, dtype, reverse, states = case
    gpu = run_case(T, B, I, H, Hp, dtype, reverse, min(0.3, H ** -0.5), states)
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        return
    for (groups, cells, rows, variant), want in ((gpu["tiling"][:4], fwd), (gpu["tiling"][4:], bwd)):
        bgroups = groups // -(-H // cells)
        tiles = -(-(-(-B // rows)) // bgroups)
        assert (rows, tiles, variant >> 8 & 1, variant >> 9 & 1) == want, gpu["tiling"]


# Time-parallel products off their tiles: widths that are no multiple of a
# tile or of a k stage, T*B no multiple of one, h0 of a batch that is no
# multiple of 32 (its own product), outputs in the halves of wider rows:
# (T, B, I, H, Hp, reverse, states)
GEMM_CASES = [
    (9, 13, 8, 40, 0, False, True),        # one partial stage each
    (5, 33, 136, 264, 0, True, True),      # k = 136: two stages and a chunk
    (17, 67, 328, 520, 0, False, False),   # more than 1024 rows, three ragged tiles per block
    (6, 250, 1096, 648, 0, False, True),   # both blocks end inside a 256-wide tile
    (4, 40, 72, 1000, 0, True, False),
    (5, 100, 200, 328, 72, False, True),   # LSTMP: Hp and 4H off the tiles
]


@pytest.mark.parametrize("T,B,I,H,Hp,reverse,states", GEMM_CASES)
def test_ragged_products(T, B, I, H, Hp, reverse, states):
    run_case(T, B, I, H, Hp, "bf16", reverse, max(I, H) ** -0.5, states)


# The fp32 products: (T, B, I, H, reverse, states)
F32_CASES = [
    (3, 5, 8, 16, False, True),       # smaller than a tile and than a stage
    (9, 7, 40, 72, True, True),       # one tile and a bit on every side
    (40, 33, 264, 136, False, False), # several tiles, split along a long k
    (7, 19, 1000, 200, False, True),
]


@pytest.mark.parametrize("T,B,I,H,reverse,states", F32_CASES)
def test_fp32_products(T, B, I, H, reverse, states):
    run_case(T, B, I, H, 0, "f32", reverse, max(I, H) ** -0.5, states)


@pytest.mark.parametrize("B,H,dtype", [(50, 648, "bf16"), (9, 264, "bf16"), (20, 200, "f32")])
def test_two_streams(B, H, dtype):
    """Layers of widths without a kernel of their own, in flight on two
    streams at once: every pass bitwise equal to the layer's pass alone, and
    no wait of a kernel timed out."""
    from paper_1907_13257_amd import Layer
    announce(f"two streams B{B} H{H} {dtype}")
    T, I = 12, 64
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(3)

    def uniform(*shape, dtype=td):
        return ((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * H ** -0.5).to(dtype)

    sets = []
    for _ in range(2):
        p = dict(W=uniform(4 * H, I), R=uniform(4 * H, H), b=uniform(4 * H, dtype=torch.float32))
        sets.append(dict(p=p, layer=Layer(T, B, I, H, 0, dtype), x=uniform(T, B, I), dy=uniform(T, B, H),
                         y=torch.empty((T, B, H), dtype=td, device="cuda"),
                         hT=torch.empty((B, H), dtype=td, device="cuda"),
                         cT=torch.empty((B, H), dtype=torch.float32, device="cuda"),
                         dx=torch.empty((T, B, I), dtype=td, device="cuda"),
                         grads={"d" + k: torch.empty(v.shape, dtype=torch.float32, device="cuda")
                                for k, v in p.items()}))

    def step(s):
        p = s["p"]
        s["layer"].forward(s["x"], p["W"], p["R"], p["b"], y=s["y"], hT=s["hT"], cT=s["cT"])
        s["layer"].backward(s["dy"], s["x"], p["W"], p["R"], s["y"], s["grads"], dx=s["dx"])

    want = []
    for s in sets:
        step(s)
        torch.cuda.synchronize()
        want.append([v.clone() for v in (s["y"], s["dx"], *s["grads"].values())])
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for st in streams:
        st.wait_stream(torch.cuda.current_stream())
    for _ in range(4):
        for s, st in zip(sets, streams):
            with torch.cuda.stream(st):
                step(s)
    torch.cuda.synchronize()
    for s, w in zip(sets, want):
        assert s["layer"].check() == 0
        for got, ref in zip((s["y"], s["dx"], *s["grads"].values()), w):
            assert torch.equal(got, ref)


@pytest.mark.parametrize("B,H", [(384, 512), (512, 512), (300, 648), (512, 1024)])
def test_row_blocks_in_flight_repeat(B, H):
    """The copies of the next row block are issued into the LDS tile whose
    fragments are being read, pair by pair; each must come after its pair's
    reads.  Passes in a row are bitwise equal at every kernel's width."""
    from paper_1907_13257_amd import Layer
    T, I = 16, 64
    announce(f"row blocks in flight B{B} H{H}")
    g = torch.Generator(device="cuda")
    g.manual_seed(B + H)

    def uniform(*shape, dtype=torch.bfloat16):
        return ((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * H ** -0.5).to(dtype)

    p = dict(W=uniform(4 * H, I), R=uniform(4 * H, H), b=uniform(4 * H, dtype=torch.float32))
    x, dy = uniform(T, B, I), uniform(T, B, H)
    lay = Layer(T, B, I, H, 0, "bf16")
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    grads = {"d" + k: torch.empty(v.shape, dtype=torch.float32, device="cuda") for k, v in p.items()}
    want = None
    for _ in range(6):
        lay.forward(x, p["W"], p["R"], p["b"], y=y)
        lay.backward(dy, x, p["W"], p["R"], y, grads, dx=dx)
        assert lay.check() == 0
        got = [v.clone() for v in (y, dx, *grads.values())]
        if want is not None:
            assert all(torch.equal(a, b) for a, b in zip(got, want))
        want = got
    lay.close()


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("T,B,H,share", [
    (3, 9, 264, "h0 in y"),       # the state carried in the last rows of y
    (4, 50, 648, "x is y"),       # the layer run in place
    (2, 20, 136, "h0 in y"),
    (3, 50, 648, "halves"),       # x and y interleaved: halves of one wider row
])
def test_inputs_inside_y(T, B, H, share, noalloc):
    """A width without a kernel of its own takes x and h0 that lie in y's
    memory (forward of two or more steps)."""
    from paper_1907_13257_amd import Layer, lstm355
    from _gpu_helpers import TOL, normwise, to_dev, to_f64
    label = f"inputs inside y T{T} B{B} H{H} {share} noalloc{int(noalloc)}"
    announce(label)
    c = layer_case(T, B, H, H, 0, "bf16", False, seed=T + B + H, scale=H ** -0.5)
    d = {k: to_dev(v) for k, v in c.items()}
    wide = share == "halves"
    buf = torch.empty((T, B, 2 * H if wide else H), dtype=torch.bfloat16, device="cuda")
    x, h0, y = d["x"], d["h0"], buf[:, :, H:] if wide else buf
    if share == "h0 in y":
        h0 = y[T - 1]
        h0.copy_(d["h0"])
    else:
        x = buf[:, :, :H]
        x.copy_(d["x"])
    hT = torch.empty((B, H), dtype=torch.bfloat16, device="cuda")
    cT = torch.empty((B, H), dtype=torch.float32, device="cuda")
    lay = Layer(T, B, H, H, 0, "bf16", ldx=2 * H if wide else 0, ldy=2 * H if wide else 0)
    if noalloc:
        lstm355.lstm_forward_noalloc(lay.handle, x, h0, d["c0"], d["W"], d["R"], d["b"], None, y, hT, cT,
                                     lay.reserve)
    else:
        lay.forward(x, d["W"], d["R"], d["b"], h0=h0, c0=d["c0"], y=y, hT=hT, cT=cT)
    assert lay.check() == 0
    ref = oracle_layer(c, 0, False)
    errs = {k: normwise(to_f64(v), ref[k]) for k, v in (("y", y.contiguous()), ("hT", hT), ("cT", cT))}
    announce(f"{label} " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()))
    assert max(errs.values()) <= TOL["bf16"]["out"], errs
    lay.close()


@pytest.mark.parametrize("Hp,states", [(0, False), (0, True), (32, False)])
def test_output_rows_spanning_more_than_2gib(Hp, states):
    """y and dy strided so far apart that their last rows lie past 2 GiB:
    every row of y still enters dR."""
    from paper_1907_13257_amd import Layer
    from _gpu_helpers import to_dev, to_f64
    T, B, I, H = 64, 32, 64, 64
    Hr, ld = Hp or H, 1 << 20
    label = f"wide rows Hp{Hp} states{int(states)}"
    announce(label)
    c = layer_case(T, B, I, H, Hp, "bf16", False, seed=Hp + states, states=states, final_grads=states,
                   scale=H ** -0.5)
    d = {k: to_dev(v) for k, v in c.items()}
    y = torch.empty((T, B, ld), dtype=torch.bfloat16, device="cuda")[:, :, :Hr]
    dy = torch.empty((T, B, ld), dtype=torch.bfloat16, device="cuda")[:, :, :Hr]
    dy.copy_(d["dy"])
    f32 = dict(dtype=torch.float32, device="cuda")
    grads = dict(dW=torch.empty((4 * H, I), **f32), dR=torch.empty((4 * H, Hr), **f32), db=torch.empty(4 * H, **f32))
    if Hp:
        grads["dP"] = torch.empty((Hp, H), **f32)
    dx = torch.empty_like(d["x"])
    lay = Layer(T, B, I, H, Hp, "bf16", ldy=ld)
    lay.forward(d["x"], d["W"], d["R"], d["b"], d["P"], d["h0"], d["c0"], y)
    lay.backward(dy, d["x"], d["W"], d["R"], y, grads, P=d["P"], h0=d["h0"], c0=d["c0"], dhT=d["dhT"],
                 dcT=d["dcT"], dx=dx)
    assert lay.check() == 0
    gpu = {k: to_f64(v.contiguous()) for k, v in dict(grads, y=y, dx=dx).items()}
    ref = oracle_layer(c, Hp, False)
    for k in ("hT", "cT", "dh0", "dc0"):   # not asked for
        gpu[k] = ref.get(k)
    check_layer(gpu, {k: v for k, v in ref.items() if v is not None}, "bf16", label)
    lay.close()


# Plain layers without a persistent tiling: more than 4096 cells, or rows of y
# strided so far apart that a tile's rows span more than 2 GiB:
# (T, B, H, dtype, ldy)
WIDE_NOALLOC_CASES = [
    (3, 3, 4104, "bf16", 0),
    (2, 33, 4608, "f32", 0),
    (2, 130, 5000, "bf16", 0),
    (2, 5, 8192, "f32", 0),
    (2, 17, 72, "bf16", (1 << 24) + 8),   # still a persistent tiling, of 16 rows
    (2, 16, 72, "bf16", 1 << 27),
]


@pytest.mark.parametrize("T,B,H,dtype,ldy", WIDE_NOALLOC_CASES)
def test_noalloc_of_layers_without_a_persistent_tiling(T, B, H, dtype, ldy):
    """lstm_forward_noalloc takes every plain layer of up to 8192 cells."""
    from paper_1907_13257_amd import Layer, lstm355
    from _gpu_helpers import TOL
    label = f"noalloc wide T{T} B{B} H{H} {dtype} ldy{ldy}"
    announce(label)
    I = 16
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(H + B)

    def uniform(*shape, dtype=td):
        return ((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * H ** -0.5).to(dtype)

    W, R, b = uniform(4 * H, I), uniform(4 * H, H), uniform(4 * H, dtype=torch.float32)
    x, h0, c0 = uniform(T, B, I), uniform(B, H), uniform(B, H, dtype=torch.float32)
    lay = Layer(T, B, I, H, 0, dtype, ldy=ldy)
    res = {}
    for mode in ("workspace", "noalloc"):
        y = torch.empty((T, B, ldy or H), dtype=td, device="cuda")[:, :, :H]
        hT, cT = torch.empty_like(h0), torch.empty_like(c0)
        if mode == "workspace":
            lay.forward(x, W, R, b, None, h0, c0, y, hT, cT)
        else:
            lstm355.lstm_forward_noalloc(lay.handle, x, h0, c0, W, R, b, None, y, hT, cT, lay.reserve)
        assert lay.check() == 0
        res[mode] = dict(y=y.double(), hT=hT.double(), cT=cT.double())
    h, c, ys = h0.double(), c0.double(), []
    Wd, Rd = W.double(), R.double()
    for t in range(T):
        i, f, u, o = (x[t].double() @ Wd.t() + h @ Rd.t() + b.double()).chunk(4, dim=1)
        c = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(u)
        h = torch.sigmoid(o) * torch.tanh(c)
        ys.append(h)
    ref = dict(y=torch.stack(ys), hT=h, cT=c)
    for mode, got in res.items():
        errs = {k: float((got[k] - ref[k]).abs().max() / ref[k].abs().max()) for k in ref}
        announce(f"{label} {mode} " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()))
        assert max(errs.values()) <= TOL[dtype]["out"], (mode, errs)
    lay.close()


@pytest.mark.parametrize("T,B,H,dtype,reverse", [(2, 3, 4104, "bf16", False), (2, 18, 4160, "f32", True)])
def test_plain_layers_wider_than_the_persistent_kernels(T, B, H, dtype, reverse):
    gpu = run_case(T, B, 24, H, 0, dtype, reverse, H ** -0.5)
    assert gpu["tiling"][3] == 2000 and gpu["tiling"][7] == 2000, gpu["tiling"]


@pytest.mark.parametrize("recurrence,variants", [("persistent", None), ("stepwise", (2000,))])
def test_recurrence_switch_at_padded_widths(recurrence, variants, monkeypatch):
    """LSTM355_RECURRENCE selects the generic kernels and the stepwise sequence
    for the widths that the XCD-local kernels pad."""
    monkeypatch.setenv("LSTM355_RECURRENCE", recurrence)
    gpu = run_case(3, 21, 40, 264, 0, "bf16", False, 264 ** -0.5)
    got = {gpu["tiling"][3], gpu["tiling"][7]}
    assert got == set(variants) if variants else not got & {1000, 1001, 2000}, gpu["tiling"]


def test_split_override_of_fp32_products(monkeypatch):
    """LSTM355_GEMM_TILE's split count reaches the fp32 products: another order
    of the sums over k, the same gradients within fp32 rounding."""
    T, B, I, H = 40, 33, 264, 136
    c = layer_case(T, B, I, H, 0, "f32", False, seed=5, scale=I ** -0.5)
    ref = oracle_layer(c, 0, False)
    got = []
    for override in ("3,1", "3,4"):
        monkeypatch.setenv("LSTM355_GEMM_TILE", override)
        announce(f"fp32 products, tile override {override}")
        got.append(run_layer_gpu(c, T, B, I, H, 0, "f32", False))
        check_layer(got[-1], ref, "f32", f"override {override}")
    assert not (got[0]["dW"] == got[1]["dW"]).all()


@pytest.mark.parametrize("dtype,tile", [("bf16", "0,1"), ("bf16", "1,3"), ("bf16", "2,1"), ("bf16", "3,4"),
                                        ("f32", "3,1"), ("f32", "3,4")])
def test_register_staged_products(dtype, tile, monkeypatch):
    """The products' kernel for operands past 2 GiB, at every tile, with and
    without splits: ragged sides, accumulation, states."""
    monkeypatch.setenv("LSTM355_GEMM_DL", "0")
    monkeypatch.setenv("LSTM355_GEMM_TILE", tile)
    run_case(9, 61, 328, 264, 0, dtype, False, 328 ** -0.5)
    run_case(5, 33, 136, 72, 40, dtype, True, 136 ** -0.5)


# Where plain layers leave the generic kernels for the stepwise sequence, and
# just before: (T, B, H, dtype, reverse), (forward stepwise, backward stepwise)
STEPWISE_RULE_CASES = [
    ((2, 33, 3000, "bf16", False), (True, False)),    # three streamed tiles
    ((2, 72, 3000, "bf16", True), (True, True)),      # five
    ((2, 40, 2048, "f32", False), (False, False)),    # two
    ((1, 40, 2048, "f32", True), (True, False)),      # one step, two streamed tiles
    ((1, 3, 4096, "bf16", False), (False, False)),    # one step, one streamed tile
    ((1, 33, 64, "f32", False), (True, False)),       # one step, the slice on chip
    ((2, 512, 1024, "f32", False), (True, True)),     # sixteen tiles on chip; eight streamed backward
    ((2, 6000, 16, "f32", True), (True, False)),      # a few cells, six tiles on chip
]


@pytest.mark.parametrize("case,stepwise", STEPWISE_RULE_CASES)
def test_stepwise_rule(case, stepwise, monkeypatch):
    T, B, H, dtype, reverse = case
    gpu = run_case(T, B, 16, H, 0, dtype, reverse, H ** -0.5)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert (gpu["tiling"][3] == 2000, gpu["tiling"][7] == 2000) == stepwise, gpu["tiling"]


@pytest.mark.parametrize("T,B,H", [(6, 128, 2560), (2, 5, 1032)])
def test_stepwise_bias_gradient_from_unrounded_sums(T, B, H, monkeypatch):
    """A plain layer's db is the fp32 sum of dz before it is rounded to bf16 on
    every path: the stepwise sequence's error is the generic kernels' within
    the order of the sums.  A column sum of the rounded dz adds one rounding of
    2^-9 per element, four to five times that error at these sizes."""
    from paper_1907_13257_amd import Layer
    g = torch.Generator(device="cuda")
    g.manual_seed(T + B)

    def uniform(*shape, dtype=torch.bfloat16):
        return ((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * H ** -0.5).to(dtype)

    I = 32
    W, R, b = uniform(4 * H, I), uniform(4 * H, H), uniform(4 * H, dtype=torch.float32)
    x, dy = (torch.randn((T, B, n), generator=g, device="cuda").to(torch.bfloat16) for n in (I, H))
    bd = b.double().requires_grad_(True)
    h = torch.zeros(B, H, dtype=torch.double, device="cuda")
    c, ys, Wd, Rd = h, [], W.double(), R.double()
    for t in range(T):
        i, f, u, o = (x[t].double() @ Wd.t() + h @ Rd.t() + bd).chunk(4, dim=1)
        c = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(u)
        h = torch.sigmoid(o) * torch.tanh(c)
        ys.append(h)
    (torch.stack(ys) * dy.double()).sum().backward()
    errs = {}
    for recurrence in ("persistent", "stepwise"):
        monkeypatch.setenv("LSTM355_RECURRENCE", recurrence)
        lay = Layer(T, B, I, H, 0, "bf16")
        y = torch.empty_like(dy)
        grads = {"d" + k: torch.empty(v.shape, dtype=torch.float32, device="cuda")
                 for k, v in dict(W=W, R=R, b=b).items()}
        lay.forward(x, W, R, b, y=y)
        lay.backward(dy, x, W, R, y, grads)
        assert lay.check() == 0
        errs[recurrence] = float((grads["db"].double() - bd.grad).norm() / bd.grad.norm())
        lay.close()
    announce(f"bias gradient T{T} B{B} H{H} " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()))
    assert errs["stepwise"] <= 1.5 * errs["persistent"], errs
