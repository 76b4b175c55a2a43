"""GPU parity of the compression-side assignment step (normalise every grid, nearest codebook
shape; paper section 4.2) against the float64 oracle.

The index is an arg-min decided by floating-point scores.  The kernel's scores are fp32-grade
(split fp16 operands, fp32 accumulation, 4 mantissa bits given to the arg-max bookkeeping), so
the comparison is: the index must equal the oracle's wherever the oracle's best and second-best
squared distances differ by more than GAP, and everywhere the distance of the chosen row must be
within GAP of the smallest one (a different but equally near row is a valid answer)."""
import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GAP = 2e-5          # squared distances are O(1): shapes and rows have unit norm


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_15742_amd import binding
    binding.lib()
    return binding


def _idx_np(idx):
    a = idx.cpu().numpy()
    return a.view(np.uint16 if a.dtype == np.int16 else np.uint32).astype(np.int64)


def _check_assignment(kb, coef, cb):
    idx, gain, bias = kb.kan_vq_assign(to_dev(coef), to_dev(cb))
    idx, gain, bias = _idx_np(idx), gain.cpu().numpy(), bias.cpu().numpy()
    shapes, g_ref, b_ref = ko.normalise_grids(coef)
    assert np.abs(gain - g_ref).max() <= 2e-6 * g_ref.max()
    assert np.abs(bias - b_ref).max() <= 2e-6 * max(np.abs(b_ref).max(), np.abs(coef).max())
    flat = shapes.reshape(-1, ko.G)
    n_bad_far, n_diff = 0, 0
    step = 256 if cb.shape[0] <= 4096 else 32            # the oracle materialises E x K x 10 doubles
    for s in range(0, flat.shape[0], step):
        d2 = ko.squared_distances(flat[s:s + step], cb)
        chosen = idx.reshape(-1)[s:s + step]
        assert (chosen >= 0).all() and (chosen < cb.shape[0]).all()
        d_chosen = d2[np.arange(d2.shape[0]), chosen]
        if d2.shape[1] > 1:
            part = np.partition(d2, 1, axis=1)
            best, second = part[:, 0], part[:, 1]
        else:
            best, second = d2[:, 0], np.full(d2.shape[0], np.inf)
        assert (d_chosen <= best + GAP).all(), float((d_chosen - best).max())
        clear = second - best > GAP
        n_bad_far += int((chosen[clear] != d2.argmin(axis=1)[clear]).sum())
        n_diff += int((chosen != d2.argmin(axis=1)).sum())
    assert n_bad_far == 0
    return idx, gain, bias, n_diff


@pytest.mark.parametrize("n_in,n_out,K", [(64, 32, 256), (37, 29, 1000), (96, 128, 65536), (5, 3, 7), (1, 1, 1),
                                          (200, 13, 70000)])
def test_assignment_matches_oracle(kb, n_in, n_out, K):
    coef, cb, k_true = synth.make_dense_grids(n_in + K, n_in, n_out, K)
    idx, gain, bias, n_diff = _check_assignment(kb, coef, cb)
    assert n_diff <= max(2, idx.size // 1000)              # near-ties are rare
    if K >= 256:
        # the layer was built from these shapes with 5 % noise: most edges find their own shape again
        assert (idx == k_true).mean() > 0.5


def test_assignment_exact_recovery_special_grids_and_r2(kb):
    rng = np.random.default_rng(3)
    cb = synth.make_shapes(rng, 4096)
    k = rng.integers(0, 4096, size=(40, 50))
    g = rng.uniform(0.05, 2.0, size=(40, 50))
    b = rng.normal(size=(40, 50))
    coef = (g[..., None] * cb[k].astype(np.float64) + b[..., None]).astype(np.float32)
    coef[0, 0] = 0.25                                     # constant grid: gain 0
    coef[0, 1] = 0.0
    idx, gain, bias = kb.kan_vq_assign(to_dev(coef), to_dev(cb))
    idx_np = _idx_np(idx)
    mask = np.ones((40, 50), dtype=bool)
    mask[0, :2] = False
    assert np.array_equal(idx_np[mask], k[mask])
    assert np.abs(gain.cpu().numpy()[mask] - g[mask]).max() < 1e-5 and gain[0, 0].item() == 0.0
    assert abs(bias[0, 0].item() - 0.25) < 1e-7
    # constant grids go to the row of smallest norm (all rows have unit norm here: any valid row)
    assert 0 <= idx_np[0, 0] < 4096
    r2 = kb.kan_vq_reconstruction_r2(to_dev(coef), to_dev(cb), idx, gain, bias)
    r2_ref = ko.r_squared(coef, cb, idx_np, gain.cpu().numpy(), bias.cpu().numpy())
    assert abs(r2 - r2_ref) < 1e-9 and r2 > 1 - 1e-6
    noisy, cb2, _ = synth.make_dense_grids(11, 64, 48, 2048, noise=0.2)
    i2, g2, b2 = kb.kan_vq_assign(to_dev(noisy), to_dev(cb2))
    r2 = kb.kan_vq_reconstruction_r2(to_dev(noisy), to_dev(cb2), i2, g2, b2)
    r2_ref = ko.r_squared(noisy, cb2, _idx_np(i2), g2.cpu().numpy(), b2.cpu().numpy())
    assert abs(r2 - r2_ref) < 1e-9 and 0.3 < r2 < 1.0


def test_assigned_layer_runs_through_the_forward_pass(kb):
    """Compress a dense layer, run the compressed layer, compare with the oracle run on the same
    compressed parameters and with the dense layer itself (close, since R^2 is high)."""
    coef, cb, _ = synth.make_dense_grids(21, 128, 96, 8192, noise=0.02)
    idx, gain, bias = kb.kan_vq_assign(to_dev(coef), to_dev(cb))
    P = synth.VQLayerParams(128, 96, 8192, cb, np.float32(1.0), _idx_np(idx).astype(np.uint16),
                            gain.cpu().numpy(), bias.cpu().numpy())
    x = synth.make_x(5, 7, 128)
    y = kb.kan_vq_layer_forward(kb.VQLayer(P), to_dev(x), path=kb.KAN_PATH_GATHER).cpu().numpy()
    y_ref = ko.vq_layer_forward(x, **P.as_dict())
    assert ko.error_report(y, y_ref)["headline"] <= 1e-5
    y_dense = ko.dense_layer_forward(coef, x)
    assert ko.error_report(y, y_dense)["headline"] < 0.15          # 2 % noise per coefficient, summed over 128 inputs


# ---- bounded search and the whole search's two forms ---------------------------------------------------


def _grids(kind, K, E, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cb = torch.randn((K, 10), generator=g, device="cuda")
    cb -= cb.mean(1, keepdim=True)
    cb /= cb.norm(dim=1, keepdim=True)
    if kind == "duplicates":
        cb[K // 2:] = cb[:K - K // 2].clone()
    if kind == "norms":
        cb *= torch.rand((K, 1), generator=g, device="cuda") * 3
    if kind == "one row":
        cb[:] = cb[:1].clone()
    if kind == "unused":           # rows that no edge was ever assigned to
        cb[torch.rand(K, generator=g, device="cuda") < 0.4] = 0.0
    if kind == "near ties":        # pairs of rows 1e-5 apart: scores that differ by less than a millionth
        cb *= 0.97 + torch.rand((K, 1), generator=g, device="cuda") * 0.06
        cb[K // 2:] = cb[:K - K // 2] + 3e-6 * torch.randn((K - K // 2, 10), generator=g, device="cuda")
    if kind == "clumps":           # cells of some hundred to some thousand shapes, most of them beyond one chunk of 512
        cb[:K // 2] = cb[torch.randint(0, 5, (K // 2,), generator=g, device="cuda")] + 0.02 * cb[:K // 2]
    k = torch.randint(0, K, (E, 1), generator=g, device="cuda")
    if kind == "one cell":
        k[:] = 5
    noise = torch.randn((E, 1, 10), generator=g, device="cuda") * (0.5 if kind == "far" else 0.05)
    gain = torch.randn((E, 1, 1), generator=g, device="cuda").abs_().mul_(0.1).add_(1e-3)
    coef = gain * (cb[k] + noise) + 0.01 * torch.randn((E, 1, 1), generator=g, device="cuda")
    if kind == "flat":
        coef[::3] = 0.0
    if kind == "no numbers":       # among the shapes that become centres of cells as well as between them
        cb[::64 * 7] = float("nan")
        cb[32::64 * 5] = float("inf")
        cb[::64 * 11] = 1e6
    return coef.contiguous(), cb.contiguous()


def _bounded_is_taken(kb, n_in, n_out, K):
    """The faster workspace is none of the whole search's: the shapes' operands, and eight bytes an edge and part of the codebook."""
    L = kb.lib()
    whole, fast = L.kan_vq_assign_workspace_bytes(K), L.kan_vq_assign_fast_workspace_bytes(n_in, n_out, K)
    return fast not in {(whole + (8 * n_in * n_out * parts if parts > 1 else 0) + 255) // 256 * 256 for parts in range(1, 33)}


@pytest.mark.parametrize("kind,K,E", [("trained", 16384, 131072), ("trained", 16421, 130901), ("trained", 50001, 60001),
                                      ("trained", 70000, 50001), ("far", 16384, 131105), ("duplicates", 16384, 131072),
                                      ("norms", 16384, 131072), ("flat", 16384, 131072), ("one cell", 16384, 131072),
                                      ("one row", 16384, 131072), ("unused", 20000, 110592)])
def test_bounded_search_finds_the_nearest_row(kb, kind, K, E):
    """Every chosen row is as near as the nearest one (fp64, on the device), and the same as the whole
    search's wherever no other row is that near."""
    coef, cb = _grids(kind, K, E, K + E)
    L = kb.lib()
    whole = torch.empty(L.kan_vq_assign_workspace_bytes(K), dtype=torch.uint8, device="cuda")
    assert _bounded_is_taken(kb, E, 1, K)
    idx, gain, bias = kb.kan_vq_assign(coef, cb)
    ref = kb.kan_vq_assign(coef, cb, ws=whole)
    assert torch.equal(gain, ref[1]) and torch.equal(bias, ref[2])
    mask = 0xffff if K <= 65536 else 0xffffffff
    a, b = idx.view(-1).long() & mask, ref[0].view(-1).long() & mask
    assert int(a.max()) < K and int(b.max()) < K
    n = coef.view(E, 10).double()
    n = n - n.mean(1, keepdim=True)
    g = n.norm(dim=1, keepdim=True)
    n = torch.where(g > 0, n / g, torch.zeros_like(n))
    c = cb.double()
    for s in range(0, E, 4096):
        d2 = (n[s:s + 4096] ** 2).sum(1, keepdim=True) - 2 * n[s:s + 4096] @ c.T + (c ** 2).sum(1)
        best, second = torch.topk(d2, 2, dim=1, largest=False).values.unbind(1)
        for x in (a, b):
            assert float((d2.gather(1, x[s:s + 4096, None])[:, 0] - best).max()) <= GAP
        clear = second - best > GAP
        assert torch.equal(a[s:s + 4096][clear], b[s:s + 4096][clear])


def _both_searches(kb, coef, cb):
    """Ids of the bounded and of the whole search."""
    E, K = coef.shape[0] * coef.shape[1], cb.shape[0]
    L = kb.lib()
    whole = torch.empty(L.kan_vq_assign_workspace_bytes(K), dtype=torch.uint8, device="cuda")
    assert _bounded_is_taken(kb, coef.shape[0], coef.shape[1], K)
    mask = 0xffff if K <= 65536 else 0xffffffff
    return [kb.kan_vq_assign(coef, cb, ws=ws)[0].view(-1).long() & mask for ws in (None, whole)]


@pytest.mark.parametrize("K,E", [(16384, 131072), (20010, 110001)])
def test_bounded_search_scores_as_well_as_the_whole_search(kb, K, E):
    """Pairs of rows whose scores differ by less than a millionth: as many edges of the bounded search as of the whole
    one get the farther row of the pair (fp64, on the device), up to four deviations of such a count."""
    coef, cb = _grids("near ties", K, E, K + E + 1)
    n = coef.view(E, 10).double()
    n = n - n.mean(1, keepdim=True)
    n /= n.norm(dim=1, keepdim=True)
    wrong = []
    for ids in _both_searches(kb, coef, cb):
        twin = torch.where(ids < K // 2, ids + K // 2, ids - K // 2)
        d2 = [((n - cb[i].double()) ** 2).sum(1) for i in (ids, twin)]
        wrong.append(int((d2[0] > d2[1]).sum()))
    assert wrong[0] <= wrong[1] + 4 * wrong[1] ** 0.5, wrong


@pytest.mark.parametrize("kind,K,E", [("trained", 16421, 130901), ("trained", 70000, 50001), ("far", 16384, 131105),
                                      ("duplicates", 16384, 131072), ("norms", 16384, 131072), ("near ties", 16384, 131072),
                                      ("flat", 16384, 131072), ("one cell", 16384, 131072), ("one row", 16384, 131072),
                                      ("unused", 16384, 131072), ("unused", 70001, 50003),
                                      # parts of a cell: 8 up to 1024 cells, 4, 2, 1 (K / 64 cells, at most 8192 parts)
                                      ("trained", 65536, 50021), ("trained", 131071, 40009), ("trained", 262144, 33013),
                                      ("trained", 300000, 32003), ("clumps", 16384, 131072), ("clumps", 65521, 50023),
                                      ("no numbers", 16384, 131072), ("duplicates", 70001, 50003), ("flat", 131071, 40009),
                                      ("no numbers", 131071, 40009), ("no numbers", 262144, 33013), ("no numbers", 300000, 32003),
                                      ("trained", 8193, 600001)])
def test_bounded_search_gives_the_ids_of_the_whole_search(kb, kind, K, E):
    """Not one id differs, whichever edges share a wave and are handed over: equal scores go to the lowest id in both,
    edges of gain 0 to the same shape, and grids that are no numbers or overflow to what the whole search gives."""
    coef, cb = _grids(kind, K, E, K + E + 2)
    odd = coef.view(E, 10)[7:1007].view(10, 100, 10)
    odd[0] = float("nan")
    odd[1, :, 3] = float("inf")
    odd[2] *= 1e30                                       # the gain overflows
    odd[3] = 0.25
    a, b = _both_searches(kb, coef, cb)
    assert torch.equal(a, b), int((a != b).sum())
    assert torch.equal(a, _both_searches(kb, coef, cb)[0])


@pytest.mark.parametrize("scale", [1e-19, 1e-21, 3e-22])
def test_bounded_search_on_grids_with_subnormal_squares(kb, scale):
    """Their normalised vectors are longer than one (the sum of squares has few bits left): still the whole search's ids."""
    coef, cb = _grids("trained", 16384, 131072, 5)
    coef *= scale
    a, b = _both_searches(kb, coef, cb)
    assert torch.equal(a, b), int((a != b).sum())


@pytest.mark.parametrize("K,E", [(16421, 131072), (1000, 3000)])
def test_shapes_of_large_norm_win_over_rows_past_the_last(kb, K, E):
    """Norms of 250 to 350 (half their square is still an fp16 number): every id is a shape, and as near as the nearest
    up to the rounding of scores of 5e4 (22 bits: 0.012, twice that for a difference, twice that for distances)."""
    coef, cb = _grids("trained", K, E, 9)
    cb *= 250 + 100 * torch.rand((K, 1), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    idx = kb.kan_vq_assign(coef, cb)[0].view(-1).long() & 0xffff
    assert int(idx.max()) < K
    n = coef.view(E, 10).double()
    n = n - n.mean(1, keepdim=True)
    n /= n.norm(dim=1, keepdim=True)
    c = cb.double()
    for s in range(0, E, 4096):
        d2 = 1.0 - 2 * n[s:s + 4096] @ c.T + (c ** 2).sum(1)
        assert float((d2.gather(1, idx[s:s + 4096, None])[:, 0] - d2.min(1).values).max()) <= 0.05


@pytest.mark.parametrize("K,E", [(1, 1), (33, 127), (257, 129), (1000, 4096), (4096, 131072), (300, 131073),
                                 (820, 262399), (820, 262400), (4096, 786431), (4096, 786432), (512, 976562), (512, 976563)])
def test_whole_search_shared_and_separate_waves(kb, K, E):
    """Operands in LDS (1, 33, 257 and 300 shapes, 512 in its last call but one), and either side of the switches between eight
    waves on 128 edges and four on 512: gathers the nearest row."""
    coef, cb = _grids("trained", K, E, K + E)
    idx, _, _ = kb.kan_vq_assign(coef, cb)
    a = idx.view(-1).long() & 0xffff
    n = coef.view(E, 10).double()
    n = n - n.mean(1, keepdim=True)
    n /= n.norm(dim=1, keepdim=True)
    c = cb.double()
    for s in range(0, E, 8192):
        d2 = 1.0 - 2 * n[s:s + 8192] @ c.T + (c ** 2).sum(1)
        assert float((d2.gather(1, a[s:s + 8192, None])[:, 0] - d2.min(1).values).max()) <= GAP


@pytest.mark.parametrize("kind", ["trained", "norms", "duplicates", "far", "no numbers"])
@pytest.mark.parametrize("K,E", [(384, 130), (512, 130), (513, 257), (8193, 127), (40000, 129), (65536, 4097), (20000, 45000)])
def test_whole_search_in_parts_and_in_one(kb, kind, K, E):
    """Shapes in LDS (384), waves that share their edges (512, 513), parts of the codebook, tiles tested by their first product
    (8,192 shapes of a part and more): the ids are those of one part (a workspace without room for several), and as near as
    the nearest row wherever the edge and its scores are numbers."""
    coef, cb = _grids(kind, K, max(E, 8192), K + E)
    coef = coef.view(-1, 10)[:E].reshape(E, 1, 10).clone()
    odd = coef.view(E, 10)[5:65].view(6, 10, 10)
    odd[0] = float("nan")
    odd[1, :, 3] = float("inf")
    odd[2] *= 1e30
    odd[3] = 0.25
    odd[4] *= 1e-21
    whole = torch.empty(kb.lib().kan_vq_assign_workspace_bytes(K), dtype=torch.uint8, device="cuda")
    mask = 0xffff if K <= 65536 else 0xffffffff
    got = kb.kan_vq_assign(coef, cb)
    one = kb.kan_vq_assign(coef, cb, ws=whole)
    assert torch.equal(got[0], one[0]) and torch.equal(got[1].nan_to_num(), one[1].nan_to_num())
    a = got[0].view(-1).long() & mask
    assert int(a.max()) < K
    n = coef.view(E, 10).double()
    n = n - n.mean(1, keepdim=True)
    g = n.norm(dim=1, keepdim=True)
    n = torch.where(g > 0, n / g, torch.zeros_like(n))
    valid = torch.ones(E, dtype=torch.bool, device="cuda")
    valid[5:65] = False                                   # (no numbers, an overflow, or a norm without bits)
    rows = torch.isfinite(cb).all(1) & (cb.abs().amax(1) < 200)        # (the others' scores are no numbers in fp16 parts)
    c = torch.where(rows[:, None], cb, torch.zeros_like(cb)).double()
    gap = GAP * max(1.0, float((c ** 2).sum(1).max()))
    for s in range(0, E, 2048):
        d2 = (n[s:s + 2048] ** 2).sum(1, keepdim=True) - 2 * n[s:s + 2048] @ c.T + (c ** 2).sum(1)
        d2[:, ~rows] = float("inf")
        far = d2.gather(1, a[s:s + 2048, None])[:, 0] - d2.min(1).values
        assert float(far[valid[s:s + 2048]].max()) <= gap


@pytest.mark.parametrize("kind,K,E", [("trained", 513, 786433), ("trained", 1000, 786433), ("trained", 65536, 49153), ("trained", 131071, 36001),
                                      ("trained", 262144, 30001), ("trained", 300000, 30001), ("clumps", 65521, 49153)])
def test_large_searches_give_the_ids_of_one_part(kb, kind, K, E):
    """Operands in LDS and waves with edges of their own (3 * 2^18 edges), and the bounded search from about where it begins for codebooks
    whose cells have eight, four, two parts and one."""
    coef, cb = _grids(kind, K, E, K + E + 2)
    whole = torch.empty(kb.lib().kan_vq_assign_workspace_bytes(K), dtype=torch.uint8, device="cuda")
    assert _bounded_is_taken(kb, E, 1, K) == (K > 1000)
    a, b = kb.kan_vq_assign(coef, cb)[0], kb.kan_vq_assign(coef, cb, ws=whole)[0]
    assert torch.equal(a, b), int((a != b).sum())
    flat = coef.view(E, 10)[:64].double()
    n = flat - flat.mean(1, keepdim=True)
    n /= n.norm(dim=1, keepdim=True)
    d2 = 1.0 - 2 * n @ cb.double().T + (cb.double() ** 2).sum(1)
    ids = a.view(-1)[:64].long() & (0xffff if K <= 65536 else 0xffffffff)
    assert float((d2.gather(1, ids[:, None])[:, 0] - d2.min(1).values).max()) <= GAP


@pytest.mark.parametrize("kind", ["trained", "duplicates", "no numbers"])
@pytest.mark.parametrize("K,E,piece", [(385, 32769, 32768), (512, 40001, 20001), (640, 65537, 32769), (640, 781249, 781248),
                                       (500, 1000001, 500001), (513, 974659, 974658), (640, 800001, 65536), (641, 229376, 229375), (819, 262080, 262079),
                                       (1500, 480001, 240001)])
def test_searches_of_few_shapes_give_the_ids_of_their_pieces(kb, kind, K, E, piece):
    """Either side of the lines between the forms of the search (operands in LDS, waves with edges of their own, shared edges):
    a call's ids, gains and biases are those of calls on pieces of its edges, which take another form; and near the nearest row."""
    coef, cb = _grids(kind, K, E, K + E + 3)
    odd = coef.view(E, 10)[E - 60:].view(6, 10, 10)
    odd[0] = float("nan")
    odd[1, :, 3] = float("inf")
    odd[2] *= 1e30
    odd[3] = 0.25
    odd[4] *= 1e-21
    got = kb.kan_vq_assign(coef, cb)
    for at in range(0, E, piece):
        part = kb.kan_vq_assign(coef[at:at + piece].clone(), cb)
        for a, b in zip(got, part):
            a, b = a.view(-1)[at:at + piece], b.view(-1)
            assert torch.equal(a, b) if a.dtype != torch.float32 else torch.equal(a.nan_to_num(), b.nan_to_num())
    if kind == "trained":
        n = coef.view(E, 10)[:8192].double()
        n = n - n.mean(1, keepdim=True)
        n /= n.norm(dim=1, keepdim=True)
        d2 = 1.0 - 2 * n @ cb.double().T + (cb.double() ** 2).sum(1)
        ids = got[0].view(-1)[:8192].long() & 0xffff
        assert float((d2.gather(1, ids[:, None])[:, 0] - d2.min(1).values).max()) <= GAP
