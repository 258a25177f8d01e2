"""Ranking on the GPU against the oracle's sort over the forms the selection
takes: row lengths at the edges of its steps and dispatch rules, both scopes,
and score distributions that are ties, signed, or unlike the sample that the
head selection brackets its thresholds with."""
import numpy as np
import pytest
import torch

from gpu_harness import lists_of, log
from oracle import rank as orank
from paper_2609_32628_amd import api

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    api.lib()


def _sampled(M):
    """Positions the head selection samples: one hashed place in each of 32,768
    (8,192 for small heads) equal strata."""
    SAMPLES = 32768 if M >= 4 * 32768 + 64 else 8192
    j = np.arange(SAMPLES, dtype=np.uint64)
    p0, p1 = j * np.uint64(M) // np.uint64(SAMPLES), (j + np.uint64(1)) * np.uint64(M) // np.uint64(SAMPLES)
    m32 = np.uint64(0xFFFFFFFF)
    x = ((j + np.uint64(1)) * np.uint64(0x9E3779B1)) & m32
    x ^= x >> np.uint64(15)
    x = (x * np.uint64(0x85EBCA77)) & m32
    x ^= x >> np.uint64(13)
    return (p0 + (((p1 - p0) * x) >> np.uint64(32))).astype(np.int64)


def _scores(kind, R, seed):
    rng = np.random.default_rng(seed)
    A = np.exp(3 * rng.standard_normal((R, R))).astype(np.float32)
    if kind == "softmax":
        A /= A.sum(axis=1, keepdims=True)
    elif kind == "constant":
        A[:] = 0.25
    elif kind == "ties":      # a spike of equal scores across every usual threshold, zeros of both signs
        A[rng.random((R, R)) < 0.6] = 1.0
        A[rng.random((R, R)) < 0.2] = 0.0
        A[rng.random((R, R)) < 0.1] = -0.0
    elif kind == "signed":
        A = rng.standard_normal((R, R)).astype(np.float32)
        A[0, :min(R, 3)] = [np.inf, -np.inf, 1e-42][:min(R, 3)]
    elif kind == "nan":       # the NaN whose bits order above every other value's, in a third of the places
        A[rng.random((R, R)) < 0.3] = np.array(0x7FFFFFFF, np.uint32).view(np.float32)
    elif kind == "unsampled-high":   # every sampled score is below every other one: all brackets miss
        A.reshape(-1)[_sampled(R * R)] = 1e-20
    elif kind == "unsampled-inside":  # all other scores lie inside the brackets: the gathered keys do not fit
        A[:] = rng.random((R, R)).astype(np.float32) * 1e-3 + 0.5
        A.reshape(-1)[_sampled(R * R)] = np.linspace(0.0, 1.0, _sampled(R * R).size, dtype=np.float32)
    return A


def _routes(buf, A, h, H, cuts):
    """How the head selection found each of head h's thresholds: "bracket" (from
    the gathered keys), "missed" (the threshold lies outside its bracket) or
    "overflow" (the gathered keys did not fit), from the brackets that the call
    left in its workspace."""
    M = A.size
    ws = buf.ws_rank.cpu().numpy()
    words = ws[:4 * H * 6144].view(np.uint32).reshape(H, 6144)[h]
    at, size = 4 * H * 6144, -(-24 * H // 256) * 256           # then thresholds, lower and upper ends
    lo, hi = (ws[at + i * size:at + i * size + 24 * H].view(np.uint64).reshape(H, 3)[h] for i in (1, 2))
    u = (A.reshape(-1) + np.float32(0)).view(np.uint32)
    img = np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.uint64)
    keys = (img << np.uint64(22)) | (np.uint64(2 ** 22 - 1) - np.arange(M, dtype=np.uint64))
    inside, out = np.zeros(M, bool), []
    for t, c in enumerate(cuts):
        if not 0 < c < M:
            out.append(None)
            continue
        mine = (keys >= lo[t]) & (keys <= hi[t])
        inside |= mine
        above = int((keys > hi[t]).sum())
        assert words[32 * t] == above
        out.append("bracket" if above < c <= above + mine.sum() else "missed")
    # its part of the class map, up to seven bytes less for the alignment
    fits = words[96] <= (M - (-h * M % 8)) // 8
    assert words[96] == inside.sum()
    return [r if r is None or fits else "overflow" for r in out]


def _check(R, scope, kind, budgets, H=2):
    num16, num8, num4, den = budgets
    log(f"ranking R={R} {scope} {kind} {budgets}")
    p = api.problem(1, H, 64, R, 7, 8)
    buf = api.alloc(p, scope)
    A = np.stack([_scores(kind, R, 10 * R + h) for h in range(H)])
    buf.A.copy_(torch.from_numpy(A[None]))
    buf.cls.fill_(0xA5)
    buf.lists.fill_(0xA5)
    api.da2_rank_assign(buf.A, p, num16, num8, num4, den, scope, buf.cls, buf.lists, buf.ws_rank)
    torch.cuda.synchronize()
    cls = buf.cls.cpu().numpy().reshape(H, R, R)
    keys, counts, order = lists_of(buf, p)
    assert np.array_equal(np.sort(order), np.arange(H * R))
    for h in range(H):
        want = orank.rank_head(np.where(np.isnan(A[h]), np.float32(np.inf), A[h]), num8, num4, den, scope, num16=num16)
        assert np.array_equal(cls[h], want), h
        if scope == "head" and R >= 182 and budgets in ROUTES.get(kind, (None, ()))[1]:
            routes = _routes(buf, A[h], h, H, np.cumsum(orank.quotas3(num16, num8, num4, den, R * R)))
            log(f"  head {h}: {routes}")
            assert all(r in (None, ROUTES[kind][0]) for r in routes)
        for a in range(R):
            row = h * R + a
            lists = orank.key_lists_all(want[a])
            assert [len(x) for x in lists] == list(counts[row, :3]) and counts[row, 3] == 0
            assert np.array_equal(keys[row, :counts[row, :3].sum()], np.concatenate(lists))


BUDGETS = (15, 10, 30, 100)
MIDDLE = [(25, 25, 25, 100), (30, 20, 20, 100), BUDGETS]
# What the kinds of scores are for, and the budgets it holds for: all but the
# sampled scores lie above every bracket, or inside the one at the median.
ROUTES = {"softmax": ("bracket", MIDDLE), "unsampled-high": ("missed", [BUDGETS, (0, 10, 30, 100)]),
          "unsampled-inside": ("overflow", [(0, 0, 50, 100)])}


@pytest.mark.parametrize("scope", ["head", "row"])
@pytest.mark.parametrize("R", [1, 2, 3, 63, 64, 65, 181, 182, 255, 256, 257, 362, 363, 513, 768, 769])
def test_row_lengths(R, scope):
    """Edges of the 256-pair steps, of the direct selection (R = 181) and of
    the larger sample (R = 363); rows start at odd addresses."""
    _check(R, scope, "softmax", BUDGETS)


@pytest.mark.parametrize("kind", ["constant", "ties", "signed", "unsampled-high", "unsampled-inside"])
@pytest.mark.parametrize("R,scope", [(150, "head"), (200, "head"), (530, "head"), (1500, "head"), (530, "row")])
def test_distributions(R, scope, kind):
    if R == 150 and kind.startswith("unsampled"):
        pytest.skip("this head is selected without a sample")
    for budgets in (BUDGETS, (0, 10, 30, 100), (0, 0, 50, 100), (1, 998, 0, 1000), (100, 0, 0, 100), (0, 0, 0, 100)):
        _check(R, scope, kind, budgets, H=1)


@pytest.mark.parametrize("R", [182, 250, 300, 362])
@pytest.mark.parametrize("budgets", MIDDLE)
def test_three_middle_thresholds_of_small_heads(R, budgets):
    """Three brackets of a sample of 8,192 together hold an eighth of the pairs;
    the gathered keys have to fit all the same."""
    _check(R, "head", "softmax", budgets, H=3)


@pytest.mark.parametrize("scope", ["head", "row"])
def test_lists_aligned_to_four_bytes(scope):
    """The lists' entries are 32 bits at most: a base between 16-byte marks."""
    R, H = 75, 2
    p = api.problem(1, H, 64, R, 7, 8)
    buf = api.alloc(p, scope)
    buf.A.copy_(torch.from_numpy(np.stack([_scores("softmax", R, h) for h in range(H)])[None]))
    raw = torch.full((buf.lists.numel() + 16,), 0xA5, dtype=torch.uint8, device="cuda")
    at = raw[4:4 + buf.lists.numel()]
    for lists in (buf.lists, at):
        lists.fill_(0xA5)
        api.da2_rank_assign(buf.A, p, *BUDGETS, scope, buf.cls, lists, buf.ws_rank)
    torch.cuda.synchronize()
    (keys, counts, order), buf.lists = lists_of(buf, p), at
    keys4, counts4, order4 = lists_of(buf, p)
    assert np.array_equal(counts, counts4) and np.array_equal(keys, keys4)
    assert np.array_equal(np.sort(order4), np.arange(H * R))
    assert (raw[:4] == 0xA5).all() and (raw[4 + buf.lists.numel():] == 0xA5).all()


@pytest.mark.parametrize("R,scope", [(20, "head"), (200, "head"), (600, "head"), (200, "row")])
def test_nan_scores(R, scope):
    """Every threshold among equal scores of the largest image, and one below."""
    for budgets in ((5, 10, 10, 100), (15, 10, 30, 100)):
        _check(R, scope, "nan", budgets, H=1)


@pytest.mark.parametrize("R,scope", [(1305, "head"), (1306, "head"), (2047, "head"), (2048, "row"), (2049, "row")])
def test_longest_rows(R, scope):
    """The first head whose gathered keys are counted in parts, the longest head
    (2^22 pairs less) and row of the register kernels, and the first row that is
    sorted in LDS."""
    _check(R, scope, "softmax", BUDGETS, H=1)
