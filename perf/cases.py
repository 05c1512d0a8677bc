"""Workloads of the pixel-level CKKS library whose speed is measured.

A case is a dict of plain values; `prepare` makes what a program holds before the call
(keys, caches, plans, pixels and ciphertexts in HBM), `run` makes one pass through the
public Python binding, `work` states what a pass cannot do without, and `exact` gives the
decoded values in 64-bit arithmetic without the library, where the ciphertexts' randomness
determines them in closed form.

Operations (key "op"):
  roundtrip  encrypt a small image, add a brightness, decrypt: one interactive request
  encrypt    pixels to ciphertexts: plain, radix cache, top-k value cache, full value cache
  filter     k x k homomorphic mean filter of an encrypted image
  decrypt    ciphertexts to pixel values
  linear     add two images, scale by a constant, rescale (a blend)
  match      squared difference of two images: sub, product, rescale, decrypt
  batch      many RGB images of different sizes through one batch plan, brightness each
  pipeline   encrypt, filter and decrypt an image in row tiles
  serve      a burst of jobs through the serving runtime
"""
import math

import numpy as np
import torch

import paper_2409_03568_amd as P
from paper_2409_03568_amd import workloads as W

# ring -> (log N, primes, prime bits, log scale): the benchmark's two parameter sets and the
# smallest and largest ring degree the library takes
RINGS = {
    "n4096": (12, 3, 36, 30),
    "n8192": (13, 4, 50, 40),
    "n2048": (11, 3, 30, 20),
    "n16384": (14, 4, 50, 40),
}
POOL = 256  # encrypted zeros of a value cache
TOPK = 64   # values of a top-k cache


def listed():
    return [
        # a thumbnail request: 16 pixels up, brightened, and back (latency and launches)
        dict(name="roundtrip_4x4_n4096", op="roundtrip", ring="n4096", H=4, W=4, b=50.0),
        # one 32x32 image at the small parameter set, encrypt and decrypt
        dict(name="roundtrip_32x32_n4096", op="roundtrip", ring="n4096", H=32, W=32, b=-12.5),
        # the benchmark image: 256x256 at N = 8192, the three ways to encrypt it
        dict(name="encrypt_plain_256x256", op="encrypt", ring="n8192", kind="plain", H=256, W=256),
        dict(name="encrypt_radix_256x256", op="encrypt", ring="n8192", kind="radix", H=256, W=256),
        dict(name="encrypt_value_256x256", op="encrypt", ring="n8192", kind="value", H=256, W=256),
        # its 3x3 mean filter and its decryption
        dict(name="filter3_256x256", op="filter", ring="n8192", H=256, W=256, k=3),
        dict(name="decrypt_256x256", op="decrypt", ring="n8192", H=256, W=256),
        # a blend of two odd-sized images at the small parameter set
        dict(name="blend_121x77_n4096", op="linear", ring="n4096", H=121, W=77, c=0.5),
        # encrypted image matching on an odd-sized pair
        dict(name="match_101x77", op="match", ring="n8192", H=101, W=77),
        # RGB images of uneven sizes through one plan, full cache, brightness per image
        dict(name="batch_8rgb", op="batch", ring="n8192", kind="full", count=8, lo=32, hi=256, shapes=3, graph=False),
        # the large image: 512x512 at N = 4096 streamed in row tiles, 5x5 filter
        dict(name="pipeline_plain_512x512", op="pipeline", ring="n4096", kind="plain", H=512, W=512, k=5, tile=64,
             streams=1),
        # a burst of serving jobs of uneven sizes
        dict(name="serve_8jobs", op="serve", ring="n8192", kind="full", count=8, lo=32, hi=128, shapes=4, k=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _image_sides(rng, most):
    """Height and width of an image of 1..most pixels, log-uniform in size, any aspect."""
    n = _log_int(rng, 1, most)
    h = max(1, min(n, _log_int(rng, 1, n)))
    return h, max(1, n // h)


def draw(rng):
    op = rng.choice(["roundtrip", "encrypt", "encrypt", "encrypt", "filter", "filter", "decrypt", "decrypt", "linear",
                     "match", "match", "batch", "pipeline", "pipeline", "serve"])
    ring = rng.choice(["n4096", "n4096", "n4096", "n8192", "n8192", "n8192", "n2048", "n16384"])
    # the largest image whose ciphertexts take no more than the listed 256x256 ones
    most = (65536 * 2 * 4 * 8192) // (2 * RINGS[ring][1] << RINGS[ring][0])
    if op == "roundtrip":
        h, w = _image_sides(rng, 1024)
        return dict(op=op, ring=ring, H=h, W=w, b=round(rng.uniform(-40, 40), 2))
    if op == "encrypt":
        h, w = _image_sides(rng, most)
        return dict(op=op, ring=ring, kind=rng.choice(["plain", "plain", "radix", "value", "full"]), H=h, W=w)
    if op == "filter":
        h, w = _image_sides(rng, most)
        return dict(op=op, ring=ring, H=h, W=w, k=rng.choice([1, 3, 3, 5, 7]))
    if op == "decrypt":
        h, w = _image_sides(rng, most)
        return dict(op=op, ring=ring, H=h, W=w)
    if op == "linear":
        h, w = _image_sides(rng, most // 4)
        return dict(op=op, ring=ring, H=h, W=w, c=round(rng.uniform(0.05, 0.95), 3))
    if op == "match":
        ring = rng.choice(["n4096", "n8192", "n8192", "n16384"])
        h, w = _image_sides(rng, {"n4096": 20000, "n8192": 8000, "n16384": 2500}[ring])
        return dict(op=op, ring=ring, H=h, W=w)
    if op == "batch":
        ring = rng.choice(["n4096", "n8192"])
        return dict(op=op, ring=ring, kind=rng.choice(["full", "full", "value", "plain"]), count=rng.randint(1, 6),
                    lo=8, hi=_log_int(rng, 16, 160), shapes=rng.randint(0, 10**6), graph=rng.choice([False, True]))
    if op == "pipeline":
        ring = rng.choice(["n4096", "n4096", "n8192"])
        side = 512 if ring == "n4096" else 160
        h, w = _log_int(rng, 16, side), _log_int(rng, 16, side)
        return dict(op=op, ring=ring, kind=rng.choice(["plain", "radix", "value"]), H=h, W=w,
                    k=rng.choice([1, 3, 5, 7]), tile=_log_int(rng, 4, 128), streams=rng.choice([1, 1, 3]))
    return dict(op="serve", ring="n8192", kind="full", count=rng.randint(1, 12), lo=16, hi=_log_int(rng, 24, 112),
                shapes=rng.randint(0, 10**6), k=rng.choice([3, 3, 5]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _shapes(case):
    """The image sizes of a batch or a burst: (height, width) each, fixed by the case."""
    r = np.random.default_rng(case["shapes"])
    h = W.log_uniform_sides(r, case["count"], case["lo"], case["hi"])
    w = W.log_uniform_sides(r, case["count"], case["lo"], case["hi"])
    return [(int(a), int(b)) for a, b in zip(h, w)]


def _inputs(case, seed):
    """Pixels (uint8, flat) and, for a batch, its segments and brightness offsets."""
    op = case["op"]
    if op == "batch":
        r = np.random.default_rng([7, seed])
        shapes = _shapes(case)
        px = [r.integers(0, 256, 3 * h * w, dtype=np.uint8) for h, w in shapes]
        seg = np.cumsum([len(p) for p in px]).astype(np.uint64)
        return np.concatenate(px), seg, r.integers(-40, 41, len(px)).astype(np.float64)
    if op == "serve":
        r = np.random.default_rng([8, seed])
        return [r.choice(256, size=s, p=W.zipf_pmf()).astype(np.uint8) for s in _shapes(case)]
    if op in ("match", "linear"):
        return W.matching_pair(seed, case["H"], case["W"])
    if op == "roundtrip":
        return W.uniform_image(seed, case["H"], case["W"])
    return W.zipf_image(seed, case["H"], case["W"])


def _gpu(px):
    return torch.from_numpy(np.ascontiguousarray(px).reshape(-1)).cuda()


def _cache(ctx, kind, px, seed):
    if kind == "radix":
        return ctx.cache_build(P.CKKS_CACHE_RADIX, base=16, digits=2, seed=W.cache_seed(seed))
    if kind == "value":
        return ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=TOPK, zero_pool=POOL, scan_px=px, seed=W.cache_seed(seed))
    if kind == "full":
        return ctx.cache_build(P.CKKS_CACHE_VALUE_FULL, zero_pool=POOL, seed=W.cache_seed(seed))
    return None


def _encrypt(s, px, out=None, first_index=0):
    if s["cache"] is None:
        return s["ctx"].encrypt_pixels(px, s["seed"], first_index=first_index, out=out)
    return s["ctx"].encrypt_cached(s["cache"], px, s["seed"], first_index=first_index, out=out)


def prepare(case, seed):
    op = case["op"]
    ctx = P.Context(*RINGS[case["ring"]])
    ctx.keygen(W.keygen_seed(seed))
    s = dict(case=case, ctx=ctx, seed=W.job_seed(seed), cache=None)
    src = _inputs(case, seed)
    if op == "roundtrip":
        s["px"] = _gpu(src)
    elif op in ("encrypt", "pipeline"):
        s["px"] = _gpu(src)
        s["cache"] = _cache(ctx, case["kind"], s["px"], seed)
        if op == "encrypt":
            s["out"] = ctx.empty(s["px"].numel())
        else:
            s["out"] = torch.empty(s["px"].numel(), dtype=torch.float64, device="cuda")
    elif op == "filter":
        s["cache"] = _cache(ctx, "radix", None, seed)
        s["img"] = _encrypt(s, _gpu(src))
        s["out"] = ctx.empty(s["img"].count, ctx.L - 1)
    elif op == "decrypt":
        s["cache"] = _cache(ctx, "full", None, seed)
        s["img"] = _encrypt(s, _gpu(src))
        s["out"] = torch.empty(s["img"].count, dtype=torch.float64, device="cuda")
    elif op in ("linear", "match"):
        s["cache"] = _cache(ctx, "full", None, seed)
        n = src[0].size
        s["a"], s["b"] = _encrypt(s, _gpu(src[0])), _encrypt(s, _gpu(src[1]), first_index=n)
        s["tmp"] = ctx.empty(n)
        s["out"] = ctx.empty(n, ctx.L - 1)
        if op == "match":
            ctx.relin_keygen((5, seed))
            s["val"] = torch.empty(n, dtype=torch.float64, device="cuda")
    elif op == "batch":
        px, s["seg"], s["b"] = src
        s["px"] = _gpu(px)
        s["cache"] = _cache(ctx, case["kind"], s["px"], seed)
        s["plan"] = P.BatchPlan(ctx, s["cache"], 8192, case["graph"])
        s["out"] = torch.empty(len(px), dtype=torch.float64, device="cuda")
    elif op == "serve":
        s["imgs"] = src
        s["cache"] = _cache(ctx, case["kind"], None, seed)
        s["server"] = P.Server(ctx, 32 << 30, max_inflight=8, filter_k=case["k"], cache=s["cache"], max_bypass=8)
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    op = case["op"]
    if op == "roundtrip":
        ct = ctx.encrypt_pixels(s["px"], s["seed"])
        ctx.add_const(ct, case["b"])
        return ct.data, ctx.decrypt_pixels(ct)
    if op == "encrypt":
        return _encrypt(s, s["px"], s["out"]).data
    if op == "filter":
        return ctx.mean_filter(s["img"], case["H"], case["W"], case["k"], out=s["out"]).data
    if op == "decrypt":
        return ctx.decrypt_pixels(s["img"], out=s["out"])
    if op == "linear":
        t = ctx.add(s["a"], s["b"], out=s["tmp"])
        t = ctx.mul_const(t, case["c"], out=t)
        return ctx.rescale(t, out=s["out"]).data
    if op == "match":
        t = ctx.sub(s["a"], s["b"], out=s["tmp"])
        t = ctx.mul(t, t, out=t)
        sq = ctx.rescale(t, out=s["out"])
        return sq.data, ctx.decrypt_pixels(sq, out=s["val"])
    if op == "batch":
        return s["plan"].run(s["px"], s["seg"], s["b"], s["seed"], out=s["out"])
    if op == "pipeline":
        return ctx.image_pipeline(s["px"], case["H"], case["W"], s["seed"], case["k"], case["tile"], case["streams"],
                                  cache=s["cache"], out=s["out"])
    srv, first, got = s["server"], 0, {}
    ids = []
    for img in s["imgs"]:
        ids.append(srv.submit(img, s["seed"], first_index=first))
        first += img.size
    while len(got) < len(ids):
        for r in srv.poll(wait_ms=1000):
            got[r["id"]] = r["pixels"]
    return [got[i] for i in ids]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    log_n, L, _, _ = RINGS[case["ring"]]
    N, op = 1 << log_n, case["op"]
    limb = 8 * N                      # one polynomial modulo one prime
    ntt = 3 * (N // 2) * log_n        # one transform: a product, a sum and a difference per butterfly
    enc = 3 * L * ntt                 # transform of v, and two back, per prime
    limbs = lambda level: min(level, 2)  # noqa: E731  limbs a decryption reads
    dec = lambda level: 2 * limbs(level) * ntt  # noqa: E731
    if op == "batch":
        n = 3 * sum(h * w for h, w in _shapes(case))
    elif op == "serve":
        n = sum(h * w for h, w in _shapes(case))
    else:
        n = case["H"] * case["W"]
    full = n * 2 * L * limb
    kind = case.get("kind", "plain")
    # ciphertexts assembled from a cache need no transforms; a top-k cache misses some pixels
    p = np.sort(W.zipf_pmf())[::-1]
    share = {"plain": 1.0, "value": float(p[TOPK:].sum()), "radix": 0.0, "full": 0.0}[kind]
    entries = {"plain": 0, "value": TOPK + POOL, "radix": 3, "full": 256 + POOL}[kind] * 2 * L * limb
    if op == "roundtrip":
        return dict(bytes=n + full + 8 * n, flops=n * (enc + dec(L)))
    if op == "encrypt":
        return dict(bytes=n + full + min(entries, 2 * full), flops=n * enc * share)
    if op == "filter":
        return dict(bytes=full + full * (L - 1) // L, flops=n * 2 * L * N * 6)
    if op == "decrypt":
        return dict(bytes=n * (2 * limbs(L) * limb + 8), flops=n * dec(L))
    if op == "linear":
        return dict(bytes=2 * full + full * (L - 1) // L, flops=n * 2 * L * N * 6)
    if op == "match":
        # transforms of the difference, of its square and of the key switching
        mul = (2 * L + L + L * L + 2 * (L + 1)) * ntt
        return dict(bytes=2 * full + full * (L - 1) // L + 8 * n, flops=n * (mul + dec(L - 1)))
    if op == "batch":
        return dict(bytes=9 * n + full + entries, flops=n * (enc * share + dec(1)))
    # pipelines and jobs: ciphertexts encrypted once and read once by the filter, its output decrypted
    return dict(bytes=9 * n + 2 * full + full * (L - 1) // L, flops=n * (enc * share + 2 * L * N * 6 + dec(1)))


# ---------------------------------------------------------------------------
# decoded values in 64 bits: with pk = (-a s + e, a) a ciphertext decrypts to
# v e + e0 + e1 s + m, whose terms the seeds determine
# ---------------------------------------------------------------------------
_U32 = np.uint64(0xFFFFFFFF)


def _mulhilo(a, b):
    a0, a1, b0, b1 = a & _U32, a >> np.uint64(32), b & _U32, b >> np.uint64(32)
    p00, p01, p10 = a0 * b0, a0 * b1, a1 * b0
    mid = (p00 >> np.uint64(32)) + (p01 & _U32) + (p10 & _U32)
    hi = a1 * b1 + (p01 >> np.uint64(32)) + (p10 >> np.uint64(32)) + (mid >> np.uint64(32))
    return hi, a * b


def _philox(t, tag, block, seed):
    """The four words of Philox4x64-10 at counters (t, tag, block, 0), broadcast; shape [..., 4]."""
    with np.errstate(over="ignore"):
        c0, c1, c2 = np.broadcast_arrays(*(np.asarray(x, dtype=np.uint64) for x in (t, tag, block)))
        c3 = np.zeros_like(c0)
        k0, k1 = (np.array(int(x) & (2**64 - 1), dtype=np.uint64) for x in seed)
        for _ in range(10):
            h0, l0 = _mulhilo(np.uint64(0xD2E7470EE14C6C93), c0)
            h1, l1 = _mulhilo(np.uint64(0xCA5A826395121157), c2)
            c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
            k0, k1 = k0 + np.uint64(0x9E3779B97F4A7C15), k1 + np.uint64(0xBB67AE8584CAA73B)
        return np.stack([c0, c1, c2, c3], axis=-1)


def _poly(t, tag, seed, N):
    return _philox(t, tag, np.arange(N // 4), seed).reshape(-1)


def _ternary(w):
    return (w >= np.uint64(0x5555555555555556)).astype(np.float64) + (w >= np.uint64(0xAAAAAAAAAAAAAAAB)) - 1.0


def _gauss(w, sigma=3.2, B=19):
    p = np.exp(-np.arange(-B, B + 1, dtype=np.float64) ** 2 / (2 * sigma * sigma))
    f = np.cumsum(p)[:-1] / p.sum()
    T = np.array([min(2**64 - 1, int(math.ldexp(x, 64))) for x in f], dtype=np.uint64)
    return np.searchsorted(T, w, side="right").astype(np.float64) - B


def _negacyclic(a, b):
    n = len(a)
    c = np.rint(np.fft.irfft(np.fft.rfft(a, 2 * n) * np.fft.rfft(b, 2 * n), 2 * n))
    return c[:n] - c[n:]


class _Exact:
    def __init__(self, ring, seed):
        log_n, _, _, log_scale = RINGS[ring]
        self.N, self.log_n, self.scale = 1 << log_n, log_n, 2.0**log_scale
        k = W.keygen_seed(seed)
        self.s, self.e = _ternary(_poly(0, 16, k, self.N)), _gauss(_poly(0, 17, k, self.N))
        self.cos = np.cos(np.pi * np.arange(self.N) / self.N)

    def value(self, x):
        return float(np.dot(x.astype(np.longdouble), self.cos.astype(np.longdouble)) / self.scale)

    def plain(self, p, t, seed):
        """Decoded value of the fresh encryption of pixel p at index t."""
        v, g0, g1 = (_poly(t, tag, seed, self.N) for tag in (1, 2, 3))
        m = np.rint(p * np.ldexp(self.cos, int(math.log2(self.scale)) + 1 - self.log_n))
        return self.value(_negacyclic(_ternary(v), self.e) + _gauss(g0) + _negacyclic(_gauss(g1), self.s) + m)

    def brightness(self, b):
        return self.value(np.rint(math.ldexp(b * self.scale, 1 - self.log_n) * self.cos))

    def cached(self, px, seed, cache_seed):
        """Decoded values of full-cache encryptions: entry of the value + pool member."""
        entry = np.array([self.plain(v, 256 + v, cache_seed) for v in range(256)])
        pool = np.array([self.plain(0, 512 + u, cache_seed) for u in range(POOL)])
        w = _philox(np.arange(px.size), 4, 0, seed)[..., 0]
        return entry[px] + pool[_mulhilo(w, np.uint64(POOL))[0].astype(np.int64)]


def exact(case, seed):
    op = case["op"]
    if op == "roundtrip":
        E, px = _Exact(case["ring"], seed), _inputs(case, seed).reshape(-1)
        add = E.brightness(case["b"])
        return None, np.array([E.plain(int(p), i, W.job_seed(seed)) + add for i, p in enumerate(px)])
    if op == "decrypt":
        E, px = _Exact(case["ring"], seed), _inputs(case, seed).reshape(-1)
        return E.cached(px, W.job_seed(seed), W.cache_seed(seed))
    if op == "batch" and case["kind"] == "full":
        px, seg, b = _inputs(case, seed)
        E = _Exact(case["ring"], seed)
        add = np.repeat([E.brightness(float(x)) for x in b], np.diff(np.concatenate([[0], seg.astype(np.int64)])))
        return E.cached(px, W.job_seed(seed), W.cache_seed(seed)) + add
    return None
