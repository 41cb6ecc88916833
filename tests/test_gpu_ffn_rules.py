"""GPU parity and times of the grouped FFN around the lines at which its size rules change over, on hand-made
dispatches."""
import numpy as np
import pytest
import torch

from paper_2512_13525_amd import binding as B
from paper_2512_13525_amd import workloads as W
from paper_2512_13525_amd.layer import to_device_bf16
from oracle import ffn

from helpers import device_time, expected_blocks

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-2                  # relative, of a layer in bf16
LARGE_MIN_TOKENS = 2048          # from here on the launch for large batches ...
ROWS128_MIN_WORKGROUPS = 176     # ... with tiled GEMMs over blocks of 128 rows from this many first-stage workgroups of them on
MAX_CUT = 8                      # ... and up to this many blocks of 64 rows as streaming items where nothing hides them


class Dispatch:
    """counts[s] requests of slot s, drawn at random from T*k."""

    def __init__(self, counts, T, k, seed=0):
        self.T, self.k, self.C = T, k, len(counts)
        self.off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        self.n = int(self.off[-1])
        assert self.n <= T * k
        self.perm = np.random.default_rng(seed).permutation(T * k)[:self.n].astype(np.int32)
        self.list = expected_blocks(self.off, B.moe_block_rows(T))
        assert self.list[0] <= B.moe_max_blocks(T, k, self.C)
        blocks = torch.zeros((B.moe_block_list_len(T, k, self.C),), dtype=torch.int32)
        blocks[:len(self.list)] = torch.from_numpy(self.list)
        self.dev = [torch.from_numpy(self.off).cuda(), torch.from_numpy(self.perm).cuda(), blocks.cuda()]

    def buffers(self, d_h, d_e):
        ws = torch.empty((B.moe_workspace_bytes(self.T, self.k, self.C, d_h, d_e, B.MOE_DTYPE_BF16),), dtype=torch.uint8,
                         device="cuda")
        B.moe_workspace_init(ws)
        return ws, torch.full((self.T * self.k, d_h), 123.0, dtype=torch.float32, device="cuda")

    def run(self, X, W13p, W2p, d_h, d_e, Yp, ws):
        B.moe_grouped_ffn(X, W13p, W2p, self.T, self.k, self.C, d_h, d_e, B.MOE_DTYPE_BF16, *self.dev, Yp, ws)

    def wide_min(self, form, d_e):
        """The option's value that makes the slots with more than 64 requests what `form` says in the launch for large batches."""
        per_block = -(-d_e // 64)
        assert form != "64 rows" or self.list[3] < self.list[2] or not self.list[2]
        return {"rule": 0, "128 rows": 1, "64 rows": max(1, int(self.list[2]) * per_block), "streaming": 1 << 20}[form]

    def form(self, d_e):
        """What the launch for large batches makes of the slots with more than 64 requests (small layers: nothing hides them)."""
        if self.list[2] <= MAX_CUT and int(self.list[2]) * -(-d_e // 64) < 64:
            return "streaming"
        return "128 rows" if int(self.list[3]) * -(-d_e // 128) >= ROWS128_MIN_WORKGROUPS else "64 rows"


def random_weights(C, d_h, d_e):
    """Packed images of N(0, 0.02) weights; which element is which does not matter to a time."""
    return (torch.empty((C, 2 * d_e, d_h), dtype=torch.bfloat16, device="cuda").normal_().mul_(0.02),
            torch.empty((C, d_h, d_e), dtype=torch.bfloat16, device="cuda").normal_().mul_(0.02))


LONG = [(130, 65, 64, 17, 200, 66)[s % 6] for s in range(150)]           # 325 blocks of 64 rows: the list wraps twice


@pytest.mark.parametrize("counts,T,k,d_h,d_e,form", [
    ([65 + s % 64 for s in range(43)] + [64, 9, 0, 33], 2048, 4, 160, 512, "64 rows"),       # 172 workgroups of 128-row blocks
    ([65 + s % 64 for s in range(44)] + [64, 9, 0, 33], 2048, 4, 160, 512, "128 rows"),      # 176
    ([65, 128, 100, 70, 64, 0, 20], 2048, 1, 160, 256, "streaming"),                         # eight blocks of 64 rows
    ([129, 192, 150, 64, 0, 20], 2048, 1, 160, 256, "64 rows"),                              # nine
    (LONG, 2048, 8, 96, 512, "128 rows"), (LONG, 2047, 8, 96, 512, None)])
def test_large_batches_by_their_own_rule(counts, T, k, d_h, d_e, form):
    """Both sides of the lines that the launch for large batches draws by itself, and of the token count from which it runs, rows
    against the oracle."""
    d = Dispatch(counts, T, k, seed=T)
    assert (d.form(d_e) if T >= LARGE_MIN_TOKENS else None) == form
    cfg = W.MoEConfig("rules", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, seed=21)
    X = W.activations(cfg)
    W13, W2 = (np.stack(w) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    want = ffn.grouped_ffn(X, W13, W2, d.off, d.perm, k)
    d13, d2 = to_device_bf16(W13), to_device_bf16(W2)
    p13, p2 = torch.empty_like(d13), torch.empty_like(d2)
    B.moe_pack_weights_bf16(d13, d2, d.C, d_h, d_e, p13, p2)
    ws, Yp = d.buffers(d_h, d_e)
    for _ in range(2):
        Yp.fill_(123.0)
        d.run(to_device_bf16(X), p13, p2, d_h, d_e, Yp, ws)
        torch.cuda.synchronize()
        got = Yp.cpu().numpy()
        assert (got[d.n:] == 123.0).all()
        num, den = np.linalg.norm(got[:d.n] - want, axis=1), np.linalg.norm(want, axis=1)
        assert (num <= 2.5 * TOL_BF16 * den + 1e-30).all(), int(np.argmax(num / den))
        assert B.moe_workspace_status(ws) == 0


@pytest.mark.parametrize("C,rows,d_h,d_e,other,limit", [(32, 128, 2048, 768, "64 rows", 0.96), (20, 78, 7168, 2048, "64 rows", 0.93),
                                                        (3, 128, 4096, 1536, "128 rows", 0.75)])
def test_line_of_the_block_size_time(C, rows, d_h, d_e, other, limit):
    """What the rule takes is faster than the other size of block (0.90, 0.86 and 0.59 of its time)."""
    d = Dispatch([rows] * C, 2048, 8)
    assert (d.list[3] * -(-d_e // 128) >= ROWS128_MIN_WORKGROUPS) == (other == "64 rows")
    w = random_weights(C, d_h, d_e)
    X = torch.empty((2048, d_h), dtype=torch.bfloat16, device="cuda").normal_()
    ws, Yp = d.buffers(d_h, d_e)
    t = []
    for form in ("rule", other):
        B.moe_workspace_set_option(ws, B.MOE_WS_OPT_WIDE_MIN_WORKGROUPS, d.wide_min(form, d_e))
        t.append(device_time(lambda: d.run(X, *w, d_h, d_e, Yp, ws), n=5))
    assert t[0] < limit * t[1], t


@pytest.mark.parametrize("rows", [36, 48])
def test_partly_filled_last_block_time(rows):
    """Slots of one full block of 32 rows and a part of another share their tiles through L2 like slots of two full blocks: no
    slower than those (1.1 allowed; with the streaming hint on the last block's loads 1.25 times as long)."""
    T, k, C, d_h, d_e = 136, 8, 17, 2048, 768
    w = random_weights(C, d_h, d_e)
    X = torch.empty((T, d_h), dtype=torch.bfloat16, device="cuda").normal_()
    t = {}
    for m in (64, rows):
        d = Dispatch([m] * C, T, k)
        ws, Yp = d.buffers(d_h, d_e)
        t[m] = device_time(lambda: d.run(X, *w, d_h, d_e, Yp, ws))
    assert t[rows] < 1.1 * t[64], t


def test_short_list_of_a_batch_that_could_have_a_long_one_time():
    """The same slots in a batch whose list could be longer than the workgroups' own blocks (128) take no longer (1.007 times,
    token rows spread over more tokens; 1.036 when they run through the loop that walks long lists)."""
    C, rows, k, d_h, d_e = 36, 100, 8, 2048, 1408
    w = random_weights(C, d_h, d_e)
    t = {}
    for T in (600, 1500, 600, 1500):
        d = Dispatch([rows] * C, T, k)
        assert d.list[0] <= 128 and (B.moe_max_blocks(T, k, C) > 128) == (T == 1500) and T * d_h * d_e < 12e9
        X = torch.empty((T, d_h), dtype=torch.bfloat16, device="cuda").normal_()
        ws, Yp = d.buffers(d_h, d_e)
        t[T] = min(t.get(T, 1e9), device_time(lambda: d.run(X, *w, d_h, d_e, Yp, ws), n=5))
    assert t[1500] < 1.025 * t[600], t


@pytest.mark.parametrize("counts,T,k,d_h,d_e,d_s,wide_min", [
    ([1, 0, 2], 2, 2, 64, 64, 128, 0),                                   # smallest; a slot without requests
    ([0, 0], 33, 1, 96, 96, 160, 0),                                     # nothing routed here, two shared blocks, odd K-steps
    ([31, 32, 33, 64, 65, 100], 383, 1, 160, 96, 32, 0),                 # last batch in blocks of 32 rows
    ([31, 32, 33, 64, 65, 100], 383, 1, 160, 96, 32, 1),                 # both sets' long slots as tiled-GEMM blocks
    ([63, 64, 65, 129, 0, 17], 384, 2, 128, 192, 64, 1),                 # first batch in blocks of 64 rows
    ([700, 5, 64, 130], 1000, 1, 64, 64, 192, 0),
    ([28 + s for s in range(100)], 1984, 4, 64, 64, 64, 0),              # bound of 224 blocks: one launch
    ([28 + s for s in range(101)], 1984, 4, 64, 64, 64, 0),              # 225: two
    ([40, 9], 50, 1, 64, 96, 64, 0),                                     # parity of the second stages differs: two
])
def test_routed_and_shared_experts_in_one_call(counts, T, k, d_h, d_e, d_s, wide_min):
    """moe_grouped_ffn_shared: both sets' rows against the oracle, twice on the same workspaces, and a list that was cut for
    another block size is refused without touching the other set."""
    d, sh = Dispatch(counts, T, k, seed=T), Dispatch([T], T, 1)
    B.moe_shared_dispatch(T, *sh.dev)
    if d.n == 0:
        d.dev[1] = torch.zeros((1,), dtype=torch.int32, device="cuda")     # an empty tensor has no address
    cfg = W.MoEConfig("shared", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, seed=5)
    X = W.activations(cfg)
    W13, W2 = (np.stack(w) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    ws13, ws2 = W.shared_expert_weights(cfg, d_s)
    want = [ffn.grouped_ffn(X, W13, W2, d.off, d.perm, k), ffn.expert_ffn(X, ws13, ws2)]
    packed = []
    for w13, w2, n, width in ((W13, W2, d.C, d_e), (ws13[None], ws2[None], 1, d_s)):
        a, b = to_device_bf16(w13), to_device_bf16(w2)
        packed.append((torch.empty_like(a), torch.empty_like(b)))
        B.moe_pack_weights_bf16(a, b, n, d_h, width, *packed[-1])
    (ws, Yp), (s_ws, Ys) = d.buffers(d_h, d_e), sh.buffers(d_h, d_s)
    X = to_device_bf16(X)
    for w in (ws, s_ws):
        B.moe_workspace_set_option(w, B.MOE_WS_OPT_WIDE_MIN_WORKGROUPS, wide_min)

    def call(s_list):
        Yp.fill_(123.0)
        Ys.fill_(123.0)
        B.moe_grouped_ffn_shared(X, *packed[0], T, k, d.C, d_h, d_e, B.MOE_DTYPE_BF16, *d.dev, Yp, ws, *packed[1], d_s,
                                 *sh.dev[:2], s_list, Ys, s_ws)
        torch.cuda.synchronize()
        return Yp.cpu().numpy(), Ys.cpu().numpy()

    def check(got, ref):
        num, den = np.linalg.norm(got - ref, axis=1), np.linalg.norm(ref, axis=1)
        assert (num <= 2.5 * TOL_BF16 * den + 1e-30).all()

    for _ in range(2):
        y, s = call(sh.dev[2])
        assert (y[d.n:] == 123.0).all()
        check(y[:d.n], want[0])
        check(s, want[1])
        assert B.moe_workspace_status(ws) == 0 and B.moe_workspace_status(s_ws) == 0
    other = sh.dev[2].clone()
    other[1] = 96 - other[1]
    y, s = call(other)
    check(y[:d.n], want[0])
    assert (s == 123.0).all() and B.moe_workspace_status(ws) == 0 and B.moe_workspace_status(s_ws) == 2


@pytest.mark.parametrize("counts,T,k,d_h,d_e", [
    ([1], 1, 1, 4, 4),                                                   # one K-step of four columns, one channel tile of four
    ([15, 0, 16, 17, 33, 1], 41, 2, 20, 36),
    ([2 + s % 30 for s in range(70)] + [0, 40], 700, 2, 68, 12),         # slots over two rounds of the scan
    ([100, 3], 103, 1, 640, 132),                                        # more K-steps than a round of the wavefronts takes
    ([0, 0, 5], 9, 1, 516, 1028),
])
def test_f32_row_tiles(counts, T, k, d_h, d_e):
    """The fp32 path at the edges of its tiles of 16 rows and 16 channels and of its K-steps of 16 columns, rows against the oracle.
    Each sum rounds once per level of a tree of at most 4 + 7 levels per 512 columns, twice over (both matrices): some 30 roundings of
    6e-8 on sums whose terms are some 3 times as large as the result."""
    d = Dispatch(counts, T, k, seed=T)
    cfg = W.MoEConfig("rows32", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, dtype="f32", seed=9)
    X = W.activations(cfg)
    W13, W2 = (np.stack(w) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    want = ffn.grouped_ffn(X, W13, W2, d.off, d.perm, k)
    ws = torch.empty((B.moe_workspace_bytes(T, k, d.C, d_h, d_e, B.MOE_DTYPE_F32),), dtype=torch.uint8, device="cuda")
    B.moe_workspace_init(ws)
    Yp = torch.full((T * k, d_h), 123.0, dtype=torch.float32, device="cuda")
    B.moe_grouped_ffn(torch.from_numpy(X).cuda(), torch.from_numpy(W13).cuda(), torch.from_numpy(W2).cuda(), T, k, d.C, d_h, d_e,
                      B.MOE_DTYPE_F32, d.dev[0], d.dev[1], None, Yp, ws)
    torch.cuda.synchronize()
    got = Yp.cpu().numpy()
    assert (got[d.n:] == 123.0).all()
    num, den = np.linalg.norm(got[:d.n] - want, axis=1), np.linalg.norm(want, axis=1)
    assert (num <= 6e-6 * den + 1e-30).all(), float((num / den).max())


@pytest.mark.parametrize("form", ["rule", "128 rows", "64 rows", "streaming"])
@pytest.mark.parametrize("counts,k,d_h,d_e", [
    ([64, 65, 0, 128, 129, 1, 192, 193, 257], 1, 64, 32),                # edges of both kinds of block; fewest K-steps
    ([66, 63, 300, 17, 130], 1, 96, 160),                                # odd numbers of K-steps: a half K-tile at the end
    ([400], 1, 224, 288),                                                # one slot: its few blocks are streaming items by the rule
    ([70 + s % 90 for s in range(65)] + [0] * 60 + [500], 4, 320, 96),   # slots beyond the first 64; groups of tiles not full
    ([s % 65 for s in range(130)], 4, 128, 64),                          # no wide slot
    ([2048], 1, 512, 1056),                                              # many blocks of one slot on every XCD
])
def test_launch_for_large_batches(counts, k, d_h, d_e, form):
    """Batches from 2048 tokens on: wide blocks of 64 and of 128 rows and streaming items found from the slots' offsets, rows
    against the oracle, three times on one workspace."""
    T = 2048
    d = Dispatch(counts, T, k, seed=len(counts))
    cfg = W.MoEConfig("large", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, seed=13)
    X = W.activations(cfg)
    W13, W2 = (np.stack(w) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    want = ffn.grouped_ffn(X, W13, W2, d.off, d.perm, k)
    d13, d2 = to_device_bf16(W13), to_device_bf16(W2)
    p13, p2 = torch.empty_like(d13), torch.empty_like(d2)
    B.moe_pack_weights_bf16(d13, d2, d.C, d_h, d_e, p13, p2)
    ws, Yp = d.buffers(d_h, d_e)
    B.moe_workspace_set_option(ws, B.MOE_WS_OPT_WIDE_MIN_WORKGROUPS, d.wide_min(form, d_e))
    for _ in range(3):
        Yp.fill_(123.0)
        d.run(to_device_bf16(X), p13, p2, d_h, d_e, Yp, ws)
        torch.cuda.synchronize()
        got = Yp.cpu().numpy()
        assert (got[d.n:] == 123.0).all()
        num, den = np.linalg.norm(got[:d.n] - want, axis=1), np.linalg.norm(want, axis=1)
        assert (num <= 2.5 * TOL_BF16 * den + 1e-30).all(), int(np.argmax(num / den))
        assert B.moe_workspace_status(ws) == 0


@pytest.mark.parametrize("counts,k", [
    ([64, 65, 0, 128, 129, 1, 192, 193, 257, 17, 16], 1),                # streaming and wide entries, light slots last in the list
    ([40 + s % 5 for s in range(100)], 4),                               # nothing wide, entries in two groups of 64
    ([(190, 66, 64, 300, 0, 30, 129, 131)[s % 8] for s in range(256)], 16),   # 768 entries: the search takes a second round
])
def test_large_batch_takes_its_rows_from_the_list(counts, k):
    """The bf16 path takes every row range from the block list, in large batches too: offsets that say something else change
    nothing (the rule's choice, blocks of 128 and of 64 rows, streaming items)."""
    T, d_h, d_e = 2048, 64, 96
    d = Dispatch(counts, T, k, seed=3)
    cfg = W.MoEConfig("list", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, seed=17)
    X = W.activations(cfg)
    W13, W2 = (np.stack(w) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    want = ffn.grouped_ffn(X, W13, W2, d.off, d.perm, k)
    d13, d2, dX = to_device_bf16(W13), to_device_bf16(W2), to_device_bf16(X)
    p13, p2 = torch.empty_like(d13), torch.empty_like(d2)
    B.moe_pack_weights_bf16(d13, d2, d.C, d_h, d_e, p13, p2)
    ws, Yp = d.buffers(d_h, d_e)
    other = torch.zeros_like(d.dev[0])
    for form in ("rule", "128 rows", "64 rows", "streaming"):
        B.moe_workspace_set_option(ws, B.MOE_WS_OPT_WIDE_MIN_WORKGROUPS, d.wide_min(form, d_e))
        Yp.fill_(123.0)
        B.moe_grouped_ffn(dX, p13, p2, T, k, d.C, d_h, d_e, B.MOE_DTYPE_BF16, other, *d.dev[1:], Yp, ws)
        torch.cuda.synchronize()
        got = Yp.cpu().numpy()
        assert (got[d.n:] == 123.0).all()
        num, den = np.linalg.norm(got[:d.n] - want, axis=1), np.linalg.norm(want, axis=1)
        assert (num <= 2.5 * TOL_BF16 * den + 1e-30).all(), int(np.argmax(num / den))
        assert B.moe_workspace_status(ws) == 0


@pytest.mark.parametrize("d_h,d_e,limit", [(2048, 2048, 0.9), (4096, 2048, 0.8)])
def test_one_long_slot_as_tiled_gemms_time(d_h, d_e, limit):
    """One slot of 500 requests is a chain of K-tiles in each of its workgroups: with two K-tiles in flight all the time it takes 0.83
    and 0.73 times as long as in streaming items (0.96 and 0.86 where the ring runs empty every second K-tile)."""
    d = Dispatch([500], 1400, 1)
    w = random_weights(1, d_h, d_e)
    X = torch.empty((1400, d_h), dtype=torch.bfloat16, device="cuda").normal_()
    ws, Yp = d.buffers(d_h, d_e)
    t = []
    for wide_min in (0, 1 << 20):
        B.moe_workspace_set_option(ws, B.MOE_WS_OPT_WIDE_MIN_WORKGROUPS, wide_min)
        t.append(device_time(lambda: d.run(X, *w, d_h, d_e, Yp, ws)))
    assert t[0] < limit * t[1], t


@pytest.mark.parametrize("T", [3584, 3585])                             # 56 requests a slot, and a few more
def test_large_batch_of_short_slots(T):
    """Both sides of the average from which a large batch takes the launch for large batches, slots of up to 300 requests and
    empty ones among them, rows against the oracle, twice on one workspace."""
    counts, k, d_h, d_e = [(40, 64, 65, 17, 0, 70, 300, 5)[s % 8] for s in range(64)], 1, 96, 160
    d = Dispatch(counts[:48] + [0] * 16, T, k, seed=T)
    cfg = W.MoEConfig("short", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, seed=23)
    X = W.activations(cfg)
    W13, W2 = (np.stack(w) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    want = ffn.grouped_ffn(X, W13, W2, d.off, d.perm, k)
    d13, d2, dX = to_device_bf16(W13), to_device_bf16(W2), to_device_bf16(X)
    p13, p2 = torch.empty_like(d13), torch.empty_like(d2)
    B.moe_pack_weights_bf16(d13, d2, d.C, d_h, d_e, p13, p2)
    ws, Yp = d.buffers(d_h, d_e)
    for _ in range(2):
        Yp.fill_(123.0)
        d.run(dX, p13, p2, d_h, d_e, Yp, ws)
        torch.cuda.synchronize()
        got = Yp.cpu().numpy()
        assert (got[d.n:] == 123.0).all()
        num, den = np.linalg.norm(got[:d.n] - want, axis=1), np.linalg.norm(want, axis=1)
        assert (num <= 2.5 * TOL_BF16 * den + 1e-30).all(), int(np.argmax(num / den))
        assert B.moe_workspace_status(ws) == 0


def test_large_batch_of_short_slots_time():
    """200 slots of 20 requests take as long at 2048 tokens as at 2047 (within 1.12; 1.36 times as long in the launch for large
    batches)."""
    t = []
    w = random_weights(200, 512, 256)
    for T in (2047, 2048):
        d = Dispatch([20] * 200, T, 4)
        X = torch.empty((T, 512), dtype=torch.bfloat16, device="cuda").normal_()
        ws, Yp = d.buffers(512, 256)
        t.append(device_time(lambda: d.run(X, *w, 512, 256, Yp, ws)))
    assert t[1] < 1.12 * t[0], t


@pytest.mark.parametrize("d_h,d_e", [(128, 192), (96, 160)])            # even and odd numbers of K-steps, a last group of two tiles
def test_threshold_keeps_slots_streaming_in_large_batches(d_h, d_e):
    """A threshold that no batch reaches keeps all slots in streaming items in the launch for large batches as in the other: the
    same bits at 2048 tokens as at 2047 (blocks of more than 32 rows; both launches then split K the same way)."""
    counts, k = [128, 100, 64, 120, 0, 192, 33, 500], 1
    d = Dispatch(counts, 2047, k, seed=31)
    cfg = W.MoEConfig("threshold", E=d.C, k=k, d_h=d_h, d_e=d_e, T=2048, n_inst=1, C=d.C, zipf_s=0.0, seed=37)
    X = to_device_bf16(W.activations(cfg))
    W13, W2 = (to_device_bf16(np.stack(w)) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    p13, p2 = torch.empty_like(W13), torch.empty_like(W2)
    B.moe_pack_weights_bf16(W13, W2, d.C, d_h, d_e, p13, p2)
    got = []
    for T in (2047, 2048):
        d.T = T
        ws, Yp = d.buffers(d_h, d_e)
        B.moe_workspace_set_option(ws, B.MOE_WS_OPT_WIDE_MIN_WORKGROUPS, 1 << 20)
        for _ in range(2):
            Yp.fill_(123.0)
            d.run(X, p13, p2, d_h, d_e, Yp, ws)
            torch.cuda.synchronize()
            got.append(Yp[:d.n].clone())
            assert (Yp[d.n:] == 123.0).all() and B.moe_workspace_status(ws) == 0
    assert all(torch.equal(got[0], g) for g in got[1:])


def test_large_by_its_work_below_2048_tokens():
    """384 to 2047 tokens take the launch for large batches where T x d_h x d_e >= 12e9: one slot of several blocks, one short, one
    without requests; alone, and with a shared expert, which is then a call of its own."""
    counts, T, k, d_h, d_e, d_s = [200, 30, 0, 70], 900, 1, 7168, 2048, 64
    assert T * d_h * d_e >= 12e9 and T * k > 56 * len(counts)
    d, sh = Dispatch(counts, T, k), Dispatch([T], T, 1)
    B.moe_shared_dispatch(T, *sh.dev)
    cfg = W.MoEConfig("work", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, seed=41)
    X = W.activations(cfg)
    W13, W2 = (np.stack(w) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    ws13, ws2 = W.shared_expert_weights(cfg, d_s)
    want = [ffn.grouped_ffn(X, W13, W2, d.off, d.perm, k), ffn.expert_ffn(X, ws13, ws2)]
    packed = []
    for w13, w2, n, width in ((W13, W2, d.C, d_e), (ws13[None], ws2[None], 1, d_s)):
        a, b = to_device_bf16(w13), to_device_bf16(w2)
        packed.append((torch.empty_like(a), torch.empty_like(b)))
        B.moe_pack_weights_bf16(a, b, n, d_h, width, *packed[-1])
    (ws, Yp), (s_ws, Ys) = d.buffers(d_h, d_e), sh.buffers(d_h, d_s)
    X = to_device_bf16(X)

    def check(got, ref):
        num, den = np.linalg.norm(got - ref, axis=1), np.linalg.norm(ref, axis=1)
        assert (num <= 2.5 * TOL_BF16 * den + 1e-30).all()

    for shared in (False, True):
        Yp.fill_(123.0)
        if shared:
            B.moe_grouped_ffn_shared(X, *packed[0], T, k, d.C, d_h, d_e, B.MOE_DTYPE_BF16, *d.dev, Yp, ws, *packed[1], d_s, *sh.dev,
                                     Ys, s_ws)
        else:
            d.run(X, *packed[0], d_h, d_e, Yp, ws)
        torch.cuda.synchronize()
        check(Yp[:d.n].cpu().numpy(), want[0])
        assert (Yp[d.n:] == 123.0).all() and B.moe_workspace_status(ws) == 0
    check(Ys.cpu().numpy(), want[1])
    assert B.moe_workspace_status(s_ws) == 0


@pytest.mark.parametrize("form,victim", [("128 rows", 2), ("64 rows", 3), ("streaming", 3), ("rule", 8)])
def test_wait_overrun_in_the_launch_for_large_batches(form, victim):
    """A block of the launch for large batches that never becomes ready: NaN in its rows, the others as they are, status bit 0, and
    after moe_workspace_init the bits of a clean run.  As for the other launches the host pre-loads the block's first-stage
    counter, so that nobody completes it, and allows a few thousand polls."""
    counts, T, k, d_h, d_e = [30, 64, 192, 129, 20, 200], 2048, 1, 192, 160
    d = Dispatch(counts, T, k, seed=2)
    entries = d.list.reshape(-1, 4)[1:]
    cfg = W.MoEConfig("late", E=d.C, k=k, d_h=d_h, d_e=d_e, T=T, n_inst=1, C=d.C, zipf_s=0.0, seed=43)
    X = to_device_bf16(W.activations(cfg))
    W13, W2 = (to_device_bf16(np.stack(w)) for w in zip(*(W.expert_weights(cfg, e) for e in range(d.C))))
    p13, p2 = torch.empty_like(W13), torch.empty_like(W2)
    B.moe_pack_weights_bf16(W13, W2, d.C, d_h, d_e, p13, p2)
    ws, Yp = d.buffers(d_h, d_e)

    def run():
        B.moe_workspace_set_option(ws, B.MOE_WS_OPT_WIDE_MIN_WORKGROUPS, d.wide_min(form, d_e))
        Yp.fill_(123.0)
        d.run(X, p13, p2, d_h, d_e, Yp, ws)
        torch.cuda.synchronize()
        assert (Yp[d.n:] == 123.0).all()
        return Yp[:d.n].cpu().numpy(), B.moe_workspace_status(ws)

    clean, status = run()
    assert status == 0
    slot, row, hi, _ = (int(v) for v in entries[victim])
    rows = np.arange(row, min(hi, row + (128 if form == "128 rows" else 64)))
    ws.view(torch.int32)[(victim + 1) * 256] = 1000
    B.moe_workspace_set_option(ws, B.MOE_WS_OPT_SPIN_LIMIT, 5000)
    got, status = run()
    assert status == 1 and np.isnan(got[rows]).all()
    others = np.setdiff1d(np.arange(d.n), rows)
    np.testing.assert_array_equal(got[others], clean[others])
    B.moe_workspace_init(ws)
    again, status = run()
    assert status == 0
    np.testing.assert_array_equal(again, clean)


def test_large_batch_refuses_a_list_of_other_blocks():
    """A list cut into blocks of 32 rows is refused by the launch for large batches: status bit 1, nothing written."""
    d = Dispatch([100, 40, 300], 2048, 1)
    X = torch.zeros((2048, 64), dtype=torch.bfloat16, device="cuda")
    w = random_weights(d.C, 64, 64)
    ws, Yp = d.buffers(64, 64)
    d.dev[2][1] = 32
    d.run(X, *w, 64, 64, Yp, ws)
    torch.cuda.synchronize()
    assert B.moe_workspace_status(ws) == 2 and (Yp == 123.0).all()
