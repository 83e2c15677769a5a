"""GPU parity of the projection GEMM (epic_gemm) against the oracle's plain
definitions (oracle.projection, float64 on the bf16 operands).

Each case names the kernel family that runs it (the host's choice by sizes, checked
before the call and, for all cases, without a GPU in test_gemm_routes.py): whole tiles of
256 or 192 rows x 256 columns, the same in equal parts of K (split), one round of whole
128- or 96-row x 128-column tiles, 256 x 128 tiles cut along K with arrival counters
(polled and fallback finish, bit-identical), streamed weights in partial sums, and whole
streamed gate|up tiles (glu).  Among them are the four projections of the 32-layer link
step at 736 rows, compile-sized row counts (checked on sampled rows), row and column tails,
tiny shapes, and m = 0.  Bars: fp32 outputs max |err| <= 1e-4 * s, s = sqrt(K) * sigma_a *
sigma_w (the spread of an output; fp32 accumulation of bf16 products leaves ~1e-6 s);
SwiGLU (bf16 output) |err| <= 2^-8 |ref| + 1e-4 s.
"""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = 2410153399
EPI = {"store": 0, "residual": 1, "swiglu": 2}


def _dev_bits(bits):
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)


def _f64(bits):
    return synth.bf16_bits_to_f32(bits).astype(np.float64)


def kernel_of(m, n, k, epi, in_layer=False):
    """The kernel family that the host chooses for these sizes, alone or in a decoder layer."""
    from paper_2410_15332_amd import epic_link as el
    f = el._lib.epic_gemm_route_name
    f.restype = ctypes.c_char_p
    return f({**EPI, "rope": 3}[epi], m, n, k, in_layer).decode()


def _run(m, n, k, epi, kernel, tag, sample=None):
    from paper_2410_15332_amd import epic_link as el
    print(f"[gpu-test] gemm m={m} n={n} k={k} {epi} {kernel}", flush=True)
    assert kernel_of(m, n, k, epi) == kernel
    sa, sw = 1.0, 1.0 / np.sqrt(k)
    a = synth.matrix_bf16(SEED, 3 * tag, (m, k), sa)
    w = synth.matrix_bf16(SEED, 3 * tag + 1, (n, k), sw)
    ws = torch.empty(el.epic_gemm_workspace_bytes(), dtype=torch.uint8, device="cuda")
    ws.fill_(0xAB)                                      # stale contents must not matter
    da, dw = _dev_bits(a), _dev_bits(w)
    c0 = None
    if epi == "swiglu":
        out = torch.full((m, n // 2), float("nan"), dtype=torch.bfloat16, device="cuda")
        el.epic_gemm(el.GEMM_SWIGLU, da, dw, act=out, workspace=ws)
    else:
        if epi == "residual":
            c0 = synth.matrix_f32(SEED, 3 * tag + 2, (m, n))
            out = torch.from_numpy(c0.copy()).cuda()
        else:
            out = torch.full((m, n), float("nan"), dtype=torch.float32, device="cuda")
        el.epic_gemm(EPI[epi], da, dw, c=out, workspace=ws)
    torch.cuda.synchronize()
    if epi == "swiglu":
        got = synth.bf16_bits_to_f32(out.view(torch.int16).cpu().numpy().view(np.uint16)).astype(np.float64)
    else:
        got = out.cpu().numpy().astype(np.float64)
    rows = np.arange(m) if sample is None else np.asarray(sample)
    ref = oracle.projection(_f64(a[rows]), _f64(w), epi, None if c0 is None else c0[rows].astype(np.float64))
    got = got[rows]
    assert np.all(np.isfinite(got)), "unwritten or non-finite outputs"
    s = np.sqrt(k) * sa * sw
    err = np.abs(got - ref)
    bound = (2.0 ** -8) * np.abs(ref) + 1e-4 * s if epi == "swiglu" else 1e-4 * s
    print(f"[gpu-test]   max|err| {err.max():.3e} (scale {s:.3f})", flush=True)
    assert np.all(err <= bound), f"max err {err.max()} at {np.unravel_index(err.argmax(), err.shape)}"
    return got


LINK = [  # the projections of the Llama-3-8B-shaped link step, 736 S rows
    (736, 6144, 4096, "store", "cut"),
    (736, 4096, 4096, "residual", "whole96"),
    (736, 28672, 4096, "swiglu", "whole192"),
    (736, 4096, 14336, "residual", "split256"),
]


def _ids(cases):
    return [f"{c[3]}_{c[0]}x{c[1]}x{c[2]}" for c in cases]


@pytest.mark.parametrize("m,n,k,epi,kernel", LINK, ids=_ids(LINK))
def test_link_step_projections(m, n, k, epi, kernel):
    _run(m, n, k, epi, kernel, tag=LINK.index((m, n, k, epi, kernel)))


BIG = [  # whole-tile rounds (compile-sized row counts), sampled rows
    (4096, 28672, 4096, "swiglu", "whole256"),
    (4100, 4224, 1024, "residual", "whole192"),   # row tail and a column tail inside a 256-wide tile
    (20480, 6144, 4096, "store", "whole256"),
]


@pytest.mark.parametrize("m,n,k,epi,kernel", BIG, ids=_ids(BIG))
def test_large_row_counts_sampled(m, n, k, epi, kernel):
    rng = np.random.default_rng(7)
    sample = sorted(set([0, 1, 255, 256, 257, m - 257, m - 256, m - 1] + rng.integers(0, m, 56).tolist()))
    _run(m, n, k, epi, kernel, tag=10 + BIG.index((m, n, k, epi, kernel)), sample=sample)


TALL = [  # whole tiles of 192 x 256 (fewer rounds x rows than 256 x 256): row and column tails
    (550, 32768, 256, "store", "whole192"),       # 3 x 128 tiles in 2 rounds of 192; last row tile 166 rows
    (600, 24448, 512, "residual", "whole192"),    # 4 x 96 tiles, last row tile 24 rows, last tile 128 columns
]


@pytest.mark.parametrize("m,n,k,epi,kernel", TALL, ids=_ids(TALL))
def test_192_row_tiles(m, n, k, epi, kernel):
    _run(m, n, k, epi, kernel, tag=60 + TALL.index((m, n, k, epi, kernel)))


WHOLE_NARROW = [  # one round of whole 96 x 128 or 128 x 128 tiles (short K): row tails (n % 128 == 0)
    (760, 4096, 2048, "store", "whole96"),        # 8 x 32 tiles of 96 rows, last row tile 88 rows
    (700, 4096, 1024, "swiglu", "whole96"),       # ffn 2048: 8 x 32 tiles of 96 x 64 outputs, last row tile 28 rows
    (800, 4096, 2048, "store", "whole128"),       # 9 x 32 tiles of 96 rows would be 288: 7 x 32 of 128, last 32 rows
    (200, 14336, 1024, "swiglu", "whole128"),     # ffn 7168: 2 x 112 tiles of 128 x 64 outputs, last row tile 72 rows
]


@pytest.mark.parametrize("m,n,k,epi,kernel", WHOLE_NARROW, ids=_ids(WHOLE_NARROW))
def test_whole_narrow_tiles(m, n, k, epi, kernel):
    _run(m, n, k, epi, kernel, tag=70 + WHOLE_NARROW.index((m, n, k, epi, kernel)))


SMALL = [
    (1, 128, 64, "store", "whole192"),            # one tile, one row, one K stage
    (28, 384, 256, "residual", "whole192"),       # two tiles, the second half past the end
    (200, 768, 512, "store", "stream"),
    (255, 384, 640, "swiglu", "stream"),          # ffn = 192
    (257, 1024, 512, "swiglu", "stream"),
    (513, 640, 1536, "residual", "split192"),
]


@pytest.mark.parametrize("m,n,k,epi,kernel", SMALL, ids=_ids(SMALL))
def test_small_and_ragged(m, n, k, epi, kernel):
    _run(m, n, k, epi, kernel, tag=20 + SMALL.index((m, n, k, epi, kernel)))


MANY = [  # streamed weights, few tiles and a long K: a tile's K stages over many workers, a plane each
    (64, 128, 14336, "residual", "stream"),       # 2 tiles of 64 columns, 56 planes each
    (16, 256, 8192, "store", "stream"),           # 4 tiles of 32 planes
    (1, 128, 4096, "swiglu", "stream"),           # one row, 2 tiles of 16 planes
    (200, 384, 1024, "swiglu", "stream"),         # two row tiles, 12 tiles of 4 planes
]


@pytest.mark.parametrize("m,n,k,epi,kernel", MANY, ids=_ids(MANY))
def test_tiles_over_many_workers(m, n, k, epi, kernel):
    _run(m, n, k, epi, kernel, tag=50 + MANY.index((m, n, k, epi, kernel)))


CUT = [  # 256 x 128 tiles cut along K: less than a round, few tiles, row tails; and whole rounds, none cut
    (736, 6144, 4096, "store", "cut"),            # 3 x 48 tiles, up to 3 parts
    (736, 6144, 4096, "residual", "cut"),
    (1700, 1280, 4096, "residual", "cut"),        # 7 x 10 tiles, last row tile 164 rows, up to 5 parts
    (200, 20480, 1536, "swiglu", "cut"),          # 160 tiles of 64 gate|up columns, one of 200 rows
    (256, 28672, 4096, "swiglu", "cut"),
    (6000, 384, 3072, "store", "cut"),            # 24 x 3 tiles, 4 or 5 parts
    (513, 128, 960, "swiglu", "cut"),             # ffn 64: 3 tiles of 15 stages over 11 workgroups
    (100, 131200, 128, "swiglu", "cut"),          # 3 rounds whole, 257 of two stages in 256 shares; 128 rows at most
    (300, 16384, 2048, "store", "cut"),           # 2 x 128 tiles: one round, nothing cut
]


@pytest.mark.parametrize("m,n,k,epi,kernel", CUT, ids=_ids(CUT))
def test_cut_tile_fallback_matches_fast_path(m, n, k, epi, kernel, monkeypatch):
    """A cut tile's last-stage owner finishes from its registers once the other parts
    have arrived; with no polls allowed (EPIC_GEMM_FINISH_POLLS=0) it always falls back
    to writing its partial and letting the last to arrive finish.  Both paths sum the
    same partials in the same K order: bit-identical outputs, each within the bar."""
    sample = None if m * n < 10000000 else sorted({0, 1, 63, 64, m // 2, m - 2, m - 1})
    fast = _run(m, n, k, epi, kernel, tag=40 + CUT.index((m, n, k, epi, kernel)), sample=sample)
    monkeypatch.setenv("EPIC_GEMM_FINISH_POLLS", "0")
    slow = _run(m, n, k, epi, kernel, tag=40 + CUT.index((m, n, k, epi, kernel)), sample=sample)
    assert np.array_equal(fast, slow)


def test_tiles_cut_into_many_parts(monkeypatch):
    """36 tiles of 224 K stages over 256 workgroups: 8 or 9 parts a tile, polled and by the
    last to arrive.  Same bar as the other cases, against float64 on the device."""
    from paper_2410_15332_amd import epic_link as el
    m, n, k = 9000, 128, 14336
    print(f"[gpu-test] gemm m={m} n={n} k={k} store cut", flush=True)
    assert kernel_of(m, n, k, "store") == "cut"
    gen = torch.Generator(device="cuda").manual_seed(SEED)
    a = torch.empty((m, k), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    w = torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0.0, k ** -0.5, generator=gen)
    ws = torch.full((el.epic_gemm_workspace_bytes(),), 0xAB, dtype=torch.uint8, device="cuda")
    out = []
    for polls in (None, "0"):
        if polls is not None:
            monkeypatch.setenv("EPIC_GEMM_FINISH_POLLS", polls)
        out.append(torch.full((m, n), float("nan"), device="cuda"))
        el.epic_gemm(el.GEMM_STORE, a, w, c=out[-1], workspace=ws)
    err = (out[0].double() - a.double() @ w.double().t().contiguous()).abs().max()
    assert float(err) <= 1e-4
    assert torch.equal(out[0], out[1])


REUSE = [(736, 6144, 4096, "residual", "cut"), (300, 1024, 512, "store", "stream")]


def test_repeated_calls_reuse_workspace():
    """Back-to-back calls with tiles cut along K and with streamed partial sums.  Each call
    has a workspace of its own, full of stale bytes: the counters are cleared by the call."""
    for _ in range(2):
        for case in REUSE:
            _run(*case, tag=30 + REUSE.index(case))


def test_empty_and_rejected_shapes():
    from paper_2410_15332_amd import epic_link as el
    ws = torch.empty(el.epic_gemm_workspace_bytes(), dtype=torch.uint8, device="cuda")
    a = torch.zeros((0, 64), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((128, 64), dtype=torch.bfloat16, device="cuda")
    c = torch.zeros((0, 128), dtype=torch.float32, device="cuda")
    el.epic_gemm(el.GEMM_STORE, a, w, c=c, workspace=ws)          # m = 0: nothing to do
    a = torch.zeros((4, 48), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((128, 48), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(el.EpicError) as e:                         # k % 64 != 0
        el.epic_gemm(el.GEMM_STORE, a, w, c=torch.zeros((4, 128), device="cuda"), workspace=ws)
    assert e.value.status == 2
    with pytest.raises(el.EpicError) as e:                         # k % 64 != 0
        el.epic_gemm(el.GEMM_STORE, a[:, :32].contiguous(), w[:, :32].contiguous(),
                     c=torch.zeros((4, 128), device="cuda"), workspace=ws)
    assert e.value.status == 2
    a = torch.zeros((4, 64), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((128, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(el.EpicError) as e:                         # workspace too small
        el.epic_gemm(el.GEMM_STORE, a, w, c=torch.zeros((4, 128), device="cuda"), workspace=ws[:1024])
    assert e.value.status == 4


STREAM = [  # weight streaming (up to 512 rows, less than a round of wide tiles): edges of its row tiles
    (32, 640, 1024, "store", "stream"),           # one full 32-row tile, 10 column tiles
    (33, 640, 1024, "residual", "stream"),        # 64-row tiles from here
    (64, 384, 4160, "swiglu", "stream"),          # 65 K stages
    (65, 4096, 1088, "store", "stream"),          # 128-row tiles, 64 columns wide
    (128, 2048, 14336, "residual", "stream"),     # ... 128 columns wide (at least 16 stages per worker)
    (129, 4096, 8192, "store", "stream"),         # two row tiles, the second with one row
    (512, 1024, 4096, "swiglu", "stream"),        # most rows
    (5, 128, 64, "swiglu", "stream"),             # one stage per tile
    (513, 128, 14336, "residual", "split192"),    # one row more: 3 wide tiles in 28 parts of K
]


@pytest.mark.parametrize("m,n,k,epi,kernel", STREAM, ids=_ids(STREAM))
def test_weight_streaming(m, n, k, epi, kernel):
    _run(m, n, k, epi, kernel, tag=80 + STREAM.index((m, n, k, epi, kernel)))


CHAINS = [  # streamed products and the longest chain of matrix instructions of a part (planes per tile)
    (500, 3072, 2048, 24, 3),           # 6144 stages over 256 workers, a chain for each of a stage's four k-slices
    (64, 16384, 2048, 32, 1),           # 8192 stages: a tile each
    (64, 4096, 14336, 56, 5),           # 14336 stages
    (256, 4096, 14336, 112, 5),         # 128-column tiles: two chains
]


@pytest.mark.parametrize("m,n,k,chain,planes", CHAINS, ids=[f"{c[0]}x{c[1]}x{c[2]}" for c in CHAINS])
def test_streamed_sums_keep_their_precision(m, n, k, chain, planes):
    """Relative 2-norm error of fp32 sums against float64.  Rounding a sum to nearest costs
    r = 2^-23 / sqrt(12) sqrt(0.541) of it (rms, mantissas log-uniform), and a matrix
    instruction rounds its running sum twice; of independent terms the sum after j of L
    instructions has j / L of the final variance.  So chains of at most c instructions
    leave r^2 c, the addition of a part's chains at most r^2, and p planes r^2 p / 2."""
    assert kernel_of(m, n, k, "store") == "stream"
    _check_error(m, n, k, chain, planes)


def _check_error(m, n, k, chain, planes):
    from paper_2410_15332_amd import epic_link as el
    gen = torch.Generator(device="cuda").manual_seed(n + m)
    a = torch.empty((m, k), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    w = torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    c = torch.empty((m, n), dtype=torch.float32, device="cuda")
    el.epic_gemm(el.GEMM_STORE, a, w, c=c,
                 workspace=torch.empty(el.epic_gemm_workspace_bytes(), dtype=torch.uint8, device="cuda"))
    ref = a.double() @ w.double().t().contiguous()
    err = float((c.double() - ref).norm() / ref.norm())
    r = 2.0 ** -23 / np.sqrt(12) * np.sqrt(0.541)
    bound = r * np.sqrt(chain + 1 + planes / 2)
    print(f"[gpu-test] {m}x{n}x{k}: error {err:.3e}, bound {bound:.3e}", flush=True)
    assert err <= bound


WIDE_CHAINS = [  # less than a round of 256-column tiles: matrix instructions per chain, chains (or planes)
    (912, 2176, 1024, "split192", 16, 5),     # 16 K stages: parts of 3 and 4
    (629, 2048, 2048, "split192", 24, 6),
    (3000, 4096, 4096, "whole192", 128, 2),
    (3000, 5120, 8192, "whole256", 256, 2),
]


@pytest.mark.parametrize("m,n,k,kernel,chain,chains", WIDE_CHAINS, ids=[f"{c[0]}x{c[1]}x{c[2]}" for c in WIDE_CHAINS])
def test_wide_tiles_keep_their_precision(m, n, k, kernel, chain, chains):
    """As above: a whole tile's chains are added one after the other to the output, which
    rounds like planes.  One chain over all of K would pass the bound (3000 x 4096 x 4096: 3.95e-7
    against 2.9e-7)."""
    assert kernel_of(m, n, k, "store") == kernel
    _check_error(m, n, k, chain, chains)


WIDE = [  # whole 256-column tiles: one K stage, an odd number, several tiles per workgroup, tails
    (2100, 8192, 64, "store", "whole192"),        # 11 x 32 tiles of one stage each
    (2048, 8192, 64, "residual", "whole256"),     # 8 x 32 tiles of one stage, a round of 256
    (2100, 8320, 192, "residual", "whole192"),    # 3 stages; the last column tile is 128 wide
    (3000, 11520, 448, "swiglu", "whole192"),     # 7 stages, ffn 5760
    (4700, 2176, 1984, "store", "whole192"),      # two chains of 15 and 16 stages; the last column tile is 128 wide
    (5000, 2048, 2112, "residual", "whole192"),   # two chains of 16 and 17 stages
    (6000, 2176, 2112, "store", "whole256"),      # two chains of 16 and 17 stages
]


@pytest.mark.parametrize("m,n,k,epi,kernel", WIDE, ids=_ids(WIDE))
def test_wide_tiles(m, n, k, epi, kernel):
    rng = np.random.default_rng(11)
    sample = sorted(set([0, 1, 127, 128, 191, 192, 255, 256, m - 2, m - 1] + rng.integers(0, m, 90).tolist()))
    _run(m, n, k, epi, kernel, tag=100 + WIDE.index((m, n, k, epi, kernel)), sample=sample)


SPLIT = [  # 256-wide tiles in equal parts of K, each an fp32 plane (few tiles, long K, over 128 rows)
    (600, 512, 4096, "residual", "split192"),     # 4 x 2 tiles of 192 rows in 8 parts of 8 stages
    (550, 640, 4160, "store", "split192"),        # 65 stages: parts of 8 and 9; the last column tile half past the end
    (700, 1280, 4096, "swiglu", "split192"),      # gate and up summed by the SwiGLU pass
    (363, 4096, 14336, "store", "split192"),      # two row tiles, 8 parts of 28 stages
    (736, 1024, 192, "store", "split192"),        # 3 stages in two parts
    (1250, 1024, 448, "residual", "split192"),    # 7 stages in three parts, last row tile 98 rows
    (700, 2048, 14336, "residual", "split256"),   # 3 x 8 tiles of 256 rows, 10 parts of 22 or 23 stages
]


@pytest.mark.parametrize("m,n,k,epi,kernel", SPLIT, ids=_ids(SPLIT))
def test_split_wide_tiles(m, n, k, epi, kernel):
    _run(m, n, k, epi, kernel, tag=110 + SPLIT.index((m, n, k, epi, kernel)))


GLU = [  # up to 128 rows of gate|up in one round of whole 64 + 64-column tiles (192 to 256 of them)
    (1, 2 * 12288, 2048),               # fewest tiles, one row; fewer K stages than tiles
    (32, 2 * 16384, 2048),              # most tiles
    (33, 2 * 12416, 2048),              # 194 tiles: no XCD order; 64-row tiles from here
    (64, 2 * 14336, 4096),
    (65, 2 * 12288, 6144),              # 128-row tiles
    (128, 2 * 14336, 4096),
]


@pytest.mark.parametrize("m,n,k", GLU, ids=[f"{m}x{n}x{k}" for m, n, k in GLU])
def test_whole_streamed_gate_up(m, n, k):
    _run(m, n, k, "swiglu", "glu", tag=120 + GLU.index((m, n, k)))
