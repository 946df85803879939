"""Performance cases: what a streaming video model asks of this library.

A case is a dict of plain values.  ``what`` names the call: ``step`` (one chunk
of a stream: evict, append, build lists, attend), ``attend`` (the attention
alone, on lists that are there), ``split`` (the attention of a chunk with few
query tiles over a long window), ``backward``, ``append``, ``topk`` (content
lists) and ``blocks`` (a step on 3-D blocks, tokens reordered on the way in and
out).  The other fields are sizes: ``batch``, ``heads``, ``tokens`` of a chunk,
``tile`` (64 or 128), ``chunks`` in the window, ``pin`` (the first chunk stays)
and ``keep``, the share of key tiles kept of the chunks that are neither pinned
nor current.  The head dimension is 128 throughout.
"""

import math

import numpy as np
import torch

import paper_2606_09150_amd as P

D = 128
SCALE = 1.0 / math.sqrt(D)
BLOCK = {128: (2, 8, 8), 64: (2, 4, 8)}   # block of a tile: frames, rows, columns
LOCAL_R = 9                               # width of the local window, in blocks


def case(name, what, batch, heads, tokens, tile, chunks, pin, keep, **more):
    return dict({"name": name, "what": what, "batch": batch, "heads": heads, "tokens": tokens, "tile": tile,
                 "chunks": chunks, "pin": pin, "keep": keep}, **more)


def listed():
    return [
        # the smallest stream step: an 8x8 grid of three frames, two heads; latency and launches
        case("step tiny", "step", 1, 2, 192, 64, 2, False, 1.0),
        # a step at 480p (three frames of 30x52), every tile kept: fewer than two rounds of workgroups
        case("step 480p dense", "step", 1, 12, 4680, 128, 4, False, 1.0),
        # the attention of a 1K step (three frames of 68x120), a layer's dominant cost
        case("attend 1k", "attend", 1, 12, 24480, 128, 5, True, 0.25),
        # a whole step at 2K (three frames of 90x160)
        case("step 2k", "step", 1, 12, 43200, 128, 4, True, 0.15),
        # one 480p frame at a time over a long window: 52 query tiles, 156 key tiles, a few heads
        case("split frames", "split", 1, 4, 1560, 128, 12, True, 1.0),
        # 64-token tiles at 480p, the last tile partial
        case("attend 64 480p", "attend", 1, 12, 4665, 64, 4, True, 0.5),
        # a training step's backward at 480p, every tile kept
        case("backward 480p dense", "backward", 1, 12, 4680, 128, 4, False, 1.0),
        # and at 1K on sparse lists
        case("backward 1k", "backward", 1, 12, 24480, 128, 5, True, 0.25),
        # a training batch of short odd chunks on 64-token tiles
        case("backward 64 ragged", "backward", 2, 6, 1531, 64, 3, True, 0.5),
        # the cache side of a 1K step
        case("append 1k", "append", 1, 12, 24480, 128, 5, True, 0.25),
        # content-adaptive lists of a 1K step
        case("topk 1k", "topk", 1, 12, 24480, 128, 5, True, 0.25),
        # a 1K step on 3-D blocks with a local window
        case("blocks 1k", "blocks", 1, 12, 24480, 128, 5, True, 0.25, frames=3, grid_h=68, grid_w=120),
    ]


MOST_FLOPS = {"backward": {128: 2.5e13, 64: 2e12}, "other": {128: 1.0e13, 64: 1e12}}


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        what = rng.choice(["step", "attend", "split", "backward", "append", "topk", "blocks"])
        tile = rng.choice([128, 128, 64])
        heads = rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
        batch = rng.choice([1, 1, 2])
        chunks = rng.randint(2, 5)
        pin = rng.random() < 0.6
        keep = rng.choice([1.0, 1.0, round(rng.uniform(0.1, 0.9), 3)])
        more = {}
        if what == "split":
            tokens, chunks = log_int(64, 2400), rng.randint(6, 32)
        elif what == "blocks":
            more = {"frames": rng.randint(2, 4), "grid_h": log_int(16, 90), "grid_w": log_int(16, 160)}
            tokens = more["frames"] * more["grid_h"] * more["grid_w"]
        else:
            tokens = log_int(128, 43200 if what in ("append", "topk") else 24480)
        c = case("", what, batch, heads, tokens, tile, chunks, pin, keep, **more)
        del c["name"]
        if what == "topk" and not 0 < budget(c) < ranked(c):
            continue                                  # every tile or none of them: no ranking
        if work(c)["flops"] <= MOST_FLOPS["backward" if what == "backward" else "other"][tile]:
            return c


# ---- inputs ---------------------------------------------------------------

def geometry(c):
    return P.uf_block_geom(c["frames"], c["grid_h"], c["grid_w"], *BLOCK[c["tile"]])


def ranked(c):
    """Key tiles of the chunks that are neither pinned nor current."""
    return (c["chunks"] - 1 - int(c["pin"])) * -(-c["tokens"] // c["tile"])


def budget(c):
    return int(c["keep"] * ranked(c))


class Draws:
    """Seeded activations: normal values, keys with a per-channel offset that all tokens of a head share."""

    def __init__(self, c, seed):
        self.shape = (c["batch"], c["tokens"], c["heads"], D)
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
        self.key_offset = 0.5 * torch.randn((c["heads"], D), generator=self.gen, device="cuda")

    def normal(self):
        return torch.randn(self.shape, generator=self.gen, device="cuda")

    def kv(self):
        k = (self.normal() + self.key_offset).to(torch.bfloat16)
        return k, self.normal().to(torch.bfloat16)

    def q(self):
        return (1.25 * self.normal()).to(torch.bfloat16)

    def do(self):
        return self.normal().to(torch.bfloat16)


def inputs(c, seed):
    """(earlier chunks' K and V, the current chunk's K and V, Q, dO) in the order in which they are drawn."""
    d = Draws(c, seed)
    earlier = [d.kv() for _ in range(c["chunks"] if c["what"] in ("step", "append", "blocks") else c["chunks"] - 1)]
    return earlier, d.kv(), d.q(), (d.do() if c["what"] == "backward" else None)


def prepare(c, seed):
    earlier, (k, v), q, do = inputs(c, seed)
    s = {"case": c, "seed": int(seed), "q": q, "k": k, "v": v, "do": do}
    tokens = c["tokens"]
    if c["what"] == "blocks":
        s["geom"] = geometry(c)
        tokens = P.uf_block_geom_tokens(s["geom"])[0]
        for name in ("qb", "kb", "vb", "ob"):
            s[name] = torch.empty((c["batch"], tokens, c["heads"], D), dtype=torch.bfloat16, device="cuda")
    s["win"] = win = P.KVWindow(c["batch"], c["heads"], tokens, c["tile"], c["chunks"], c["pin"])
    if c["what"] == "blocks":
        win.set_block_geom(c["frames"], c["grid_h"], c["grid_w"], *BLOCK[c["tile"]])
    for ek, ev in earlier:
        if c["what"] == "blocks":
            permute(s, ek, s["kb"])
            permute(s, ev, s["vb"])
            ek, ev = s["kb"], s["vb"]
        win.append(ek, ev)
    if c["what"] in ("attend", "split", "backward", "topk"):
        win.append(k, v)
        win.build_lists(seed, c["keep"])
    if c["what"] == "backward":
        s["o"], s["lse"] = win.attention(q)
    return s


def permute(s, src, dst, inverse=0):
    P.uf_block_permute(s["geom"], s["case"]["batch"], s["case"]["heads"], src, dst, inverse)


def lists(win):
    counts, idx, mask = win.lists_views()
    return {"counts": counts, "idx": idx, "mask": mask}


def run(s):
    c, win = s["case"], s["win"]
    what = c["what"]
    if what == "attend":
        o, lse = win.attention(s["q"])
        return {"o": o, "lse": lse}
    if what == "split":
        o, lse = win.attention(s["q"], split="tail")
        return {"o": o, "lse": lse}
    if what == "backward":
        dq, dk, dv = win.attention_bwd(s["q"], s["o"], s["lse"], s["do"])
        return {"dq": dq, "dk": dk, "dv": dv}
    if what == "topk":
        win.build_topk_lists(s["q"], budget(c))
        return lists(win)
    if what == "step":
        win.evict(1)
        win.append(s["k"], s["v"])
        win.build_lists(s["seed"], c["keep"])
        o, lse = win.attention(s["q"])
        return dict(lists(win), o=o, lse=lse)
    if what == "append":
        win.evict(1)
        win.append(s["k"], s["v"])
        slot, _ = win.logical(win.info().n_live - 1)
        means = win.kmean_view()
        pages = win.pool[:means.storage_offset() * 4].view(torch.int16).view(c["chunks"], -1)
        return {"pages": pages[slot], "pooled": means[slot]}
    win.evict(1)
    permute(s, s["k"], s["kb"])
    permute(s, s["v"], s["vb"])
    permute(s, s["q"], s["qb"])
    win.append(s["kb"], s["vb"])
    win.build_lists(s["seed"], c["keep"], local_r=LOCAL_R)
    win.attention(s["qb"], out=s["ob"], lse=False)
    o = torch.empty_like(s["q"])
    permute(s, s["ob"], o, 1)
    return dict(lists(win), o=o)


# ---- what a pass cannot do without ------------------------------------------

def near(n, block, half):
    """Sum of the products of the sizes of blocks at most ``half`` apart, over n places cut into blocks."""
    size = [min(block, n - i) for i in range(0, n, block)]
    return sum(a * sum(size[max(0, i - half):i + half + 1]) for i, a in enumerate(size))


def work(c):
    B, H, L, T, n = c["batch"], c["heads"], c["tokens"], c["tile"], c["chunks"]
    forced = 1 + int(c["pin"])
    nt = -(-L // T)
    chunk = 2 * B * H * L * D                        # bytes of one bf16 tensor of a chunk
    rows = B * H * nt
    list_bytes = rows * (4 + 4 * n * nt + 4 * -(-n * nt // 32))
    pooled = 4 * rows * D
    pairs = B * H * L * L * (forced + c["keep"] * (n - forced))
    forward = {"bytes": 2 * chunk + 2 * n * chunk + 4 * B * H * L, "flops": 4 * D * pairs}
    append = {"bytes": 4 * chunk + pooled, "flops": B * H * L * D}
    if c["what"] in ("attend", "split"):
        return forward
    if c["what"] == "append":
        return append
    if c["what"] == "step":
        return {"bytes": forward["bytes"] + append["bytes"] + list_bytes, "flops": forward["flops"] + append["flops"]}
    if c["what"] == "topk":
        return {"bytes": chunk + pooled * (n - forced) + list_bytes, "flops": B * H * L * D + 2 * D * rows * ranked(c)}
    if c["what"] == "backward":
        return {"bytes": 3 * chunk + 4 * B * H * L + 2 * n * chunk + 2 * chunk + 4 * n * chunk, "flops": 10 * D * pairs}
    _, bh, bw = BLOCK[T]
    local = near(c["grid_h"], bh, LOCAL_R // 2) * near(c["grid_w"], bw, LOCAL_R // 2) / (c["grid_h"] * c["grid_w"]) ** 2
    return {"bytes": forward["bytes"] + append["bytes"] + 4 * 2 * chunk, "flops": forward["flops"] * local + append["flops"]}


def tolerance(c):
    if c["what"] == "topk":
        return "exact"
    if c["what"] == "append":
        return {"rel": 1e-6, "max": 1e-5}
    # bf16 weights and, of the forward, bf16 outputs: 1.2e-3 to 3.5e-3 off the 64-bit result
    return {"rel": 1e-2, "max": 0.1}


# ---- the same in 64 bits, from the definitions --------------------------------

def splitmix64(z):
    z = z + np.uint64(0x9E3779B97F4A7C15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def drawn_keep(c, seed, seqs, n_tiles):
    """bool [B, H, query tile, chunk, key tile]: the seeded draw of each earlier chunk's key tiles."""
    B, H = c["batch"], c["heads"]
    fields = (np.arange(B).reshape(B, 1, 1, 1, 1), np.arange(H).reshape(1, H, 1, 1, 1), np.array(seqs[-1]),
              np.arange(n_tiles).reshape(1, 1, n_tiles, 1, 1), np.array(seqs).reshape(1, 1, 1, -1, 1),
              np.arange(n_tiles).reshape(1, 1, 1, 1, n_tiles))
    with np.errstate(over="ignore"):
        x = np.array(int(seed), dtype=np.uint64)
        for f in fields:
            x = splitmix64(x ^ f.astype(np.uint64))
    keep = (x >> np.uint64(32)).astype(np.float64) < math.floor(c["keep"] * 2.0 ** 32)
    keep[:, :, :, -1] = True
    if c["pin"]:
        keep[:, :, :, 0] = True
    return torch.from_numpy(keep).cuda()


def blocks_of(c):
    """(block of each token, bool [block, block] within the local window)."""
    bt, bh, bw = BLOCK[c["tile"]]
    nh, nw = -(-c["grid_h"] // bh), -(-c["grid_w"] // bw)
    t, y, x = np.meshgrid(np.arange(c["frames"]), np.arange(c["grid_h"]), np.arange(c["grid_w"]), indexing="ij")
    of = ((t // bt) * nh + y // bh) * nw + x // bw
    j = np.arange(-(-c["frames"] // bt) * nh * nw)
    row, col = (j // nw) % nh, j % nw
    local = (abs(row[:, None] - row) <= LOCAL_R // 2) & (abs(col[:, None] - col) <= LOCAL_R // 2)
    return torch.from_numpy(of.reshape(-1)).cuda(), torch.from_numpy(local).cuda()


def exact(c, seed):
    if c["what"] == "topk":
        return None
    earlier, current, q, do = inputs(c, seed)
    B, H, L, T, what = c["batch"], c["heads"], c["tokens"], c["tile"], c["what"]
    if what == "append":
        k = torch.nn.functional.pad(current[0].double(), (0, 0, 0, 0, 0, -L % T))
        n = torch.full((k.shape[1] // T,), T, dtype=torch.float64, device="cuda")
        n[-1] = L - (len(n) - 1) * T
        return {"pages": None, "pooled": k.view(B, -1, T, H, D).sum(2).permute(0, 2, 1, 3) / n[:, None]}
    seqs = list(range(len(earlier) + 1))
    if what in ("step", "blocks"):                   # the oldest chunk that is not pinned has left
        del seqs[1 if c["pin"] else 0]
    window = [(earlier + [current])[s] for s in seqs]
    tile_of, local = blocks_of(c) if what == "blocks" else (torch.arange(L, device="cuda") // T, None)
    n_tiles = int(tile_of.max()) + 1
    keep = drawn_keep(c, seed, seqs, n_tiles)
    if local is not None:
        keep &= local[None, None, :, None, :]
    keep = keep[..., tile_of].flatten(3)             # per key token: [B, H, query tile, chunks * L]
    qh = q.double()
    o = torch.empty((B, L, H, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, H, L), dtype=torch.float64, device="cuda")
    dq = torch.empty_like(o)
    dk = torch.empty((len(window), B, L, H, D), dtype=torch.float64, device="cuda") if do is not None else None
    dv = torch.empty_like(dk) if do is not None else None
    step = max(64, int(2.5e8) // (len(window) * L))
    for b in range(B):
        for h in range(H):
            K = torch.cat([k[b, :, h].double() for k, _ in window])
            V = torch.cat([v[b, :, h].double() for _, v in window])
            gk, gv = torch.zeros_like(K), torch.zeros_like(V)
            for r in range(0, L, step):
                rows = slice(r, min(L, r + step))
                Q = qh[b, rows, h].contiguous()
                s = (Q @ K.T).mul_(SCALE).masked_fill_(~keep[b, h][tile_of[rows]], -math.inf)
                l = torch.logsumexp(s, 1)
                p = s.sub_(l[:, None]).exp_()
                lse[b, h, rows] = l
                out = p @ V
                o[b, rows, h] = out
                if do is not None:
                    g = do[b, rows, h].double()
                    gv += p.T @ g
                    ds = (g @ V.T).sub_((g * out).sum(1, keepdim=True)).mul_(p)
                    dq[b, rows, h] = ds @ K * SCALE
                    gk += ds.T @ Q * SCALE
                    del ds
                del s, p
            if do is not None:
                dk[:, b, :, h] = gk.view(len(window), L, D)
                dv[:, b, :, h] = gv.view(len(window), L, D)
    if what == "backward":
        return {"dq": dq, "dk": dk, "dv": dv}
    if what in ("attend", "split"):
        return {"o": o, "lse": lse}
    none = {"counts": None, "idx": None, "mask": None}
    return dict(none, o=o) if what == "blocks" else dict(none, o=o, lse=lse)
