"""What this library's speed is measured on: decode calls as programs make them.

A case is a decoder (lexicon, 4-gram LM, parameters) and one pass of calls on
it: a whole batch at once, or streams fed chunk by chunk.  The shapes are those
of the repository's workloads (1k / 20k / 125k words, beams 8..256, 1..1024
streams, 10-frame calls) and the regimes around them: one live stream, odd beams,
ragged batches, raw scores, recombination by maximum, an external fusion scorer,
calls that allocate nothing.

The lexicon and the LM are a program's model: they depend on the case's sizes
alone.  The log-probabilities, the lengths and the fusion scorer are the inputs
and come from the seed.
"""

import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2603_14002_amd as lb

BLANK, SEP, CLASSES = 0, 40, 41
LN10 = 2.302585092994045684

# what a case leaves unsaid: the App. E hyper-parameters of the repository's workloads
DEFAULTS = dict(batch=1, frames=50, chunk=0, ragged=False, beam=32, subbeams=3, words=20_000, ngrams=1_000_000,
                sigma=1.5, fusion="none", interval=0, top_f=0, marks=0, merge="lse", raw=False, width=256,
                noalloc=False)
ALPHA, BETA, GAMMA, OMEGA, PHI, THETA, LAMBDA = 0.6, 1.5, 1.0, 0.5, 1.2, 22.0, 4.0
FUSION_LO, FUSION_HI = -10.0, -0.5


def listed():
    return [
        # one short utterance, a small vocabulary: the smallest whole call
        dict(name="utterance-tiny", frames=50, beam=8, words=1_000, ngrams=5_000, sigma=1.0),
        # one live speaker: 25 calls of two 80-ms frames, the regime where a call's own cost shows
        dict(name="live-speaker", frames=50, chunk=2, beam=64, fusion="synthetic", interval=10),
        # one utterance at the widest beam, from raw scores, every hypothesis fused and closed by a mark:
        # how the paper decodes (one utterance at a time, fusion every 10 frames)
        dict(name="utterance-wide", frames=400, beam=256, words=125_000, ngrams=10_000_000, raw=True,
             fusion="synthetic", interval=10, marks=3),
        # a batch of utterances at a small beam
        dict(name="batch-k32", batch=64, frames=200, beam=32, sigma=1.0, fusion="synthetic", interval=20),
        # offline transcription at a medium beam: as many utterances as compute units
        dict(name="batch-k64", batch=256, frames=500, beam=64, words=125_000, ngrams=50_000_000,
             fusion="synthetic", interval=16, top_f=16),
        # the largest: offline transcription at the widest beam, two utterances per compute unit
        dict(name="batch-k256", batch=512, frames=500, beam=256, words=125_000, ngrams=50_000_000,
             fusion="synthetic", interval=16, top_f=32),
        # a server's thousand live streams, ten frames a call
        dict(name="streams-k64", batch=1024, frames=100, chunk=10, beam=64, words=125_000, ngrams=50_000_000,
             fusion="synthetic", interval=8),
        # utterances of many lengths, an odd beam, four sub-beams, the paper's recombination by maximum
        dict(name="ragged-k100-max", batch=100, frames=333, ragged=True, beam=100, subbeams=4, merge="max"),
        # somewhat more wide-beam utterances than compute units
        dict(name="ragged-k200", batch=300, frames=250, ragged=True, beam=200, words=125_000, ngrams=10_000_000,
             fusion="synthetic", interval=16, top_f=32),
        # many utterances at a small beam, raw scores, no fusion, output rows of an odd width
        dict(name="crowd-k16-raw", batch=1500, frames=100, beam=16, subbeams=2, raw=True, width=75),
        # the caller's own fusion scorer: the round trip every 20 frames and at the end
        dict(name="external-k32", batch=24, frames=120, beam=32, sigma=1.0, fusion="external", interval=20, top_f=8),
        # a serving loop that may not allocate: eight streams, eight frames a call
        dict(name="noalloc-k64", batch=8, frames=48, chunk=8, beam=64, words=125_000, ngrams=10_000_000,
             fusion="synthetic", interval=8, noalloc=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    words, ngrams = rng.choice([(1_000, 5_000), (20_000, 1_000_000), (125_000, 10_000_000), (125_000, 10_000_000)])
    c = dict(words=words, ngrams=ngrams, sigma=round(rng.uniform(1.0, 1.6), 2), subbeams=rng.choice([1, 2, 3, 3, 3, 4]))
    c["beam"] = log_int(4, 256)
    c["batch"] = log_int(1, 1024)
    c["frames"] = log_int(20, 500)
    most = 20_000_000  # stream-frames x beam: a third of the largest listed case
    while c["batch"] * c["frames"] * c["beam"] > most:
        key = rng.choice(["batch", "frames", "beam"])
        c[key] = max(1, int(c[key] * 0.7))
    c["ragged"] = rng.random() < 0.5
    if rng.random() < 0.3:
        c["chunk"] = rng.randint(max(1, c["frames"] // 40), 20)
    c["merge"] = rng.choice(["lse", "lse", "lse", "max"])
    c["raw"] = rng.random() < 0.3
    fusion = rng.choice(["none", "synthetic", "synthetic", "synthetic", "external"])
    if fusion != "none":
        c.update(fusion=fusion, interval=rng.randint(7, 24), top_f=rng.choice([0, max(1, c["beam"] // rng.randint(2, 8))]))
        if fusion == "synthetic" and rng.random() < 0.3:
            c["marks"] = rng.randint(1, 3)
    calls = -(-c["frames"] // c["chunk"]) if c.get("chunk") else 1
    c["width"] = 256 if calls * c["batch"] * c["beam"] < 2_000_000 else 64
    if c["frames"] <= 150 and rng.random() < 0.3:
        c["width"] = rng.randint(70, 150)
    return c


def full(case):
    return SimpleNamespace(**{**DEFAULTS, **{k: v for k, v in case.items() if k != "name"}})


# ---- the model: lexicon and LM


@functools.lru_cache(maxsize=None)
def lexicon(words):
    rng = np.random.default_rng([1, words])
    length = rng.integers(1, (12 if words > 50_000 else 8) + 1, size=words)
    offsets = np.zeros(words + 1, np.int32)
    np.cumsum(length, out=offsets[1:])
    return SimpleNamespace(n_words=words, offsets=offsets, phonemes=rng.integers(1, 40, size=int(offsets[-1])).astype(np.int32))


@functools.lru_cache(maxsize=2)
def language_model(words, ngrams):
    """Orders 2..4 take 40 / 35 / 25 % of the n-grams past the unigrams: a context drawn from the order below
    (1 % of the bigrams' contexts are <s>) and a word.  rows[n-1]: the sorted keys context row * vocab + word."""
    g = torch.Generator(device="cuda").manual_seed(ngrams)
    vocab, bos, unk = words + 3, words, words + 2

    def uniform(n, lo, hi):
        return (torch.rand(n, generator=g, device="cuda") * (hi - lo) + lo).cpu().numpy()

    rest = ngrams - vocab
    ids = [np.arange(vocab, dtype=np.int32)[:, None]]
    logp, bo, rows = [uniform(vocab, -4.0, -0.5)], [uniform(vocab, -1.0, 0.0)], [None]
    logp[0][bos] = -99.0
    below = torch.arange(vocab, device="cuda", dtype=torch.int32)[:, None]
    for n, share in ((2, 0.40), (3, 0.35), (4, 0.25)):
        count = int(rest * share)
        context = torch.randint(0, words if n == 2 else below.shape[0], (count,), generator=g, device="cuda")
        if n == 2:
            context[torch.rand(count, generator=g, device="cuda") < 0.01] = bos
        key = torch.unique(context * vocab + torch.randint(0, words, (count,), generator=g, device="cuda"))
        below = torch.cat([below[key // vocab], (key % vocab).to(torch.int32)[:, None]], dim=1)
        ids.append(below.cpu().numpy())
        rows.append(key.cpu().numpy())
        logp.append(uniform(len(key), -4.0, -0.5))
        if n < 4:
            bo.append(uniform(len(key), -1.0, 0.0))
    del below, key, context
    torch.cuda.empty_cache()
    return SimpleNamespace(vocab_size=vocab, bos=bos, unk=unk, ids=ids, logp=logp, bo=bo, rows=rows)


# ---- the inputs of a seed


def spoken(lex, lm, count, rng):
    """Word ids [len(count), max(count)] that follow the LM: each next word is an explicit continuation of the
    longest context that has one, else any word."""
    B, V = len(count), lm.vocab_size
    ctx = [np.full(B, lm.bos, np.int64), np.full(B, -1, np.int64), np.full(B, -1, np.int64)]  # rows, orders 1..3
    out = np.zeros((B, int(max(count))), np.int64)
    for k in range(out.shape[1]):
        w = rng.integers(0, lex.n_words, size=B)
        for n in (2, 3, 4):
            lo, hi = (np.searchsorted(lm.rows[n - 1], (ctx[n - 2] + d) * V) for d in (0, 1))
            has = (ctx[n - 2] >= 0) & (hi > lo)
            at = lo + (rng.random(B) * (hi - lo)).astype(np.int64)
            w = np.where(has, lm.rows[n - 1][np.where(has, at, 0)] % V, w)
        out[:, k] = w
        after = [w]
        for n in (2, 3):
            key = ctx[n - 2] * V + w
            at = np.minimum(np.searchsorted(lm.rows[n - 1], key), len(lm.rows[n - 1]) - 1)
            after.append(np.where((ctx[n - 2] >= 0) & (lm.rows[n - 1][at] == key), at, -1))
        ctx = after
    return out


def targets(c, lex, lm, rng):
    """The class of every frame [batch, frames]: 3..15 words and then silence for utterances, speech without end for
    streams; a symbol lasts 1 + Geometric frames after a Geometric run of blanks."""
    count = rng.integers(3, 16, size=c.batch) if not c.chunk else np.full(c.batch, c.frames // 8 + 1)
    said = spoken(lex, lm, count, rng)
    out = np.zeros((c.batch, c.frames), np.int64)
    for b in range(c.batch):
        symbols = np.concatenate([np.append(lex.phonemes[lex.offsets[w]:lex.offsets[w + 1]], SEP) for w in said[b, :count[b]]])
        blanks = rng.geometric(0.4, size=len(symbols)) - 1
        blanks[1:] = np.maximum(blanks[1:], symbols[1:] == symbols[:-1])
        runs = np.stack([blanks, rng.geometric(0.4, size=len(symbols))], 1).ravel()
        frames = np.repeat(np.stack([np.zeros_like(symbols), symbols], 1).ravel(), runs)[:c.frames]
        out[b, :len(frames)] = frames
    return out


def inputs(c, seed):
    """(scores float32 [batch, frames, 41] on the GPU, lengths int32 [batch], seed of the fusion scorer)."""
    rng = np.random.default_rng([2, seed])
    lex, lm = lexicon(c.words), language_model(c.words, c.ngrams)
    target = torch.from_numpy(targets(c, lex, lm, rng)).cuda()
    x = torch.randn(c.batch, c.frames, CLASSES, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")
    x = (x * c.sigma).scatter_add_(2, target[..., None], torch.full_like(target, 4.0, dtype=torch.float32)[..., None])
    if not c.raw:
        x = torch.log_softmax(x.double(), dim=2).float()
    lengths = np.full(c.batch, c.frames, np.int32)
    if c.ragged:
        lengths = rng.integers(c.frames // 2, c.frames + 1, size=c.batch).astype(np.int32)
    return x, lengths, int(rng.integers(0, 2**63))


def external_table(vocab, fusion_seed):
    """The caller's stand-in scorer for the external round trip: a log-probability per word."""
    g = torch.Generator(device="cuda").manual_seed(fusion_seed % 2**62)
    return torch.rand(vocab, generator=g, device="cuda") * -8.0 - 0.5


def marks_of(c, lm):
    return [lm.bos + 1, 7, 11][:c.marks]  # </s> and two words of the vocabulary


def prepare(case, seed):
    c = full(case)
    lex, lm = lexicon(c.words), language_model(c.words, c.ngrams)
    x, lengths, fusion_seed = inputs(c, seed)
    source = dict(none=lb.LB_FUSION_NONE, synthetic=lb.LB_FUSION_SYNTH_BIGRAM, external=lb.LB_FUSION_EXTERNAL)[c.fusion]
    p = SimpleNamespace(beam=c.beam, subbeams=c.subbeams, alpha=ALPHA, beta=BETA, gamma=GAMMA, omega=OMEGA, phi=PHI, theta=THETA,
                        lam=LAMBDA, fusion_interval=c.interval, fusion_top_f=c.top_f, fusion_lo=FUSION_LO, fusion_hi=FUSION_HI,
                        max_words_out=c.width)
    params = lb.make_params(p, max_batch=c.batch, max_frames=c.frames, fusion_source=source, fusion_seed=fusion_seed,
                            merge=lb.LB_MERGE_MAX if c.merge == "max" else lb.LB_MERGE_LOGSUMEXP,
                            input=lb.LB_INPUT_LOGITS if c.raw else lb.LB_INPUT_LOGPROBS, eos_count=c.marks,
                            eos_ids=tuple(marks_of(c, lm) + [0] * (3 - c.marks)))
    s = SimpleNamespace(c=c, decoder=lb.Decoder(lex, lm, params), calls=[])
    step = c.chunk or c.frames
    for lo in range(0, c.frames, step):
        n = min(step, c.frames - lo)
        flags = (lb.LB_BEGIN if lo == 0 else 0) | (lb.LB_END if lo + n == c.frames else 0)
        s.calls.append((x[:, lo:lo + n].contiguous(), torch.from_numpy(np.clip(lengths - lo, 0, n).astype(np.int32)).cuda(), n, flags))
    s.hyps = torch.empty(len(s.calls), c.batch, c.beam, c.width, dtype=torch.int32, device="cuda")
    s.scores = torch.empty(len(s.calls), c.batch, c.beam, dtype=torch.float32, device="cuda")
    if c.fusion == "external":
        s.table = external_table(lm.vocab_size, fusion_seed)
        s.words = torch.empty(c.batch, c.beam, c.subbeams, c.width, dtype=torch.int32, device="cuda")
        s.n_words = torch.empty(c.batch, c.beam, c.subbeams, dtype=torch.int32, device="cuda")
    return s


def run(s):
    """Every call of the pass; the ranked words and scores that each call returned."""
    c, handle = s.c, s.decoder.handle
    for k, (x, lengths, n, flags) in enumerate(s.calls):
        if c.noalloc:
            lb.lb_decode_batch_noalloc(handle, x, lengths, c.batch, n, flags, None, s.hyps[k], s.scores[k])
            continue
        while lb.lb_decode_batch(handle, x, lengths, c.batch, n, flags, None, s.hyps[k], s.scores[k]) == lb.LB_NEED_FUSION:
            lb.lb_fusion_request(handle, s.words, s.n_words, None)
            scores = torch.where(s.words >= 0, s.table[s.words.clamp(min=0)], 0.0).sum(-1)
            lb.lb_fusion_scores(handle, scores, None)
    return {"hyps": s.hyps, "scores": s.scores}


def work(case):
    """Log-probabilities in, ranked rows and scores out; per hypothesis and frame two log-sum-exps in 64 bits (~35
    operations each) and about six extensions of four additions and a comparison."""
    c = full(case)
    calls = -(-c.frames // (c.chunk or c.frames))
    return {"bytes": c.batch * (c.frames * CLASSES * 4 + 4 * calls) + calls * c.batch * c.beam * (c.width + 1) * 4,
            "flops": 100 * c.batch * c.frames * c.beam}


def tolerance(case):
    """Scores are sums in 64 bits given out in 32: they agree to the last place.  Two hypotheses whose totals are that
    close may change places, and the words of their rows with them."""
    return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}


# ---- the same decode in plain numpy, 64 bits


def splitmix64(x):
    m = 2**64 - 1
    z = (x + 0x9E3779B97F4A7C15) & m
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return z ^ (z >> 31)


class Plain:
    """One utterance at a time.  A hypothesis is a list [ab, anb, pt, trie node, last symbol, prefix id, parent's prefix
    id, sub-beams]; a sub-beam is (score, history) and a history (words, context rows of orders 1..3, fusion score)."""

    def __init__(self, c, fusion_seed):
        self.c, self.lm, self.seed = c, language_model(c.words, c.ngrams), fusion_seed
        self.children, self.spelled = [{}], [[]]
        lex = lexicon(c.words)
        phonemes, offsets = lex.phonemes.tolist(), lex.offsets.tolist()
        for w in range(lex.n_words):
            node = 0
            for ph in phonemes[offsets[w]:offsets[w + 1]]:
                at = self.children[node].get(ph)
                if at is None:
                    at = self.children[node][ph] = len(self.children)
                    self.children.append({})
                    self.spelled.append([])
                node = at
            self.spelled[node].append(w)
        self.table = external_table(self.lm.vocab_size, fusion_seed).cpu().numpy() if c.fusion == "external" else None

    def merge(self, x, y):
        if x < y:
            x, y = y, x
        if y == -math.inf or self.c.merge == "max":
            return x
        return x + math.log1p(math.exp(y - x))

    def bigram(self, a, b):
        return FUSION_LO + (FUSION_HI - FUSION_LO) * ((splitmix64(self.seed ^ ((a << 32) | b)) >> 48) / 65536.0)

    def query(self, hist, words):
        """(log10 P of each word after hist, its rows as an order-2 and order-3 entry, -1 where absent)."""
        lm, V = self.lm, self.lm.vocab_size
        w = np.asarray(words, np.int64)
        lp, found = lm.logp[0][w].astype(np.float64), []
        for n in (2, 3, 4):
            ctx = hist[1][n - 2]
            if ctx < 0:
                found.append(np.full(len(w), -1))
                continue
            lp = float(lm.bo[n - 2][ctx]) + lp
            key = ctx * V + w
            at = np.minimum(np.searchsorted(lm.rows[n - 1], key), len(lm.rows[n - 1]) - 1)
            hit = lm.rows[n - 1][at] == key
            lp = np.where(hit, lm.logp[n - 1][at].astype(np.float64), lp)
            found.append(np.where(hit, at, -1))
        return lp, found[0], found[1]

    def completed(self, subs, words):
        O, H, got = self.c.subbeams, len(words), []
        for j, (L, hist) in enumerate(subs):
            lp, r2, r3 = self.query(hist, words)
            s = L + OMEGA * LN10 * lp
            for h in np.argsort(-s, kind="stable")[:O]:
                got.append((-float(s[h]), j * H + int(h), hist, words[h], int(r2[h]), int(r3[h])))
        got.sort(key=lambda g: g[:2])
        out = []
        for s, _, hist, w, r2, r3 in got[:O]:
            if -s < -got[0][0] - LAMBDA:
                break
            last = hist[0][-1] if hist[0] else self.lm.bos
            out.append((-s, (hist[0] + (w,), (w, r2, r3), hist[2] + self.bigram(last, w))))
        return out

    def fuse(self, hyps, final):
        c = self.c
        if c.fusion == "none":
            return
        chosen = hyps
        if not final and 0 < c.top_f < len(hyps):
            chosen = sorted(hyps, key=lambda h: -(h[2] + h[7][0][0]))[:c.top_f]
        for h in chosen:
            subs = []
            for _, hist in h[7]:
                if self.table is not None:
                    f = float(self.table[list(hist[0])].sum()) if hist[0] else 0.0
                else:
                    f = hist[2]
                    if final and c.marks:
                        f += max(self.bigram(hist[0][-1] if hist[0] else self.lm.bos, m) for m in marks_of(c, self.lm))
                subs.append((PHI * f, hist))
            h[7] = sorted(subs, key=lambda s: -s[0])

    def frame(self, hyps, d, ids):
        c = self.c
        by_id = {h[5]: h for h in hyps}
        merged = set()
        stays = []
        for h in hyps:
            ab, anb, pt, node, last, me, up, subs = h
            ab2 = pt + d[BLANK]
            anb2 = anb + d[last] if last else -math.inf
            parent = by_id.get(up)
            if parent is not None:
                base = parent[0] if parent[4] == last else parent[2]
                anb2 = self.merge(anb2, base + d[last] + (GAMMA if last == SEP else BETA))
                merged.add((up, last))
            pt2 = self.merge(ab2, anb2)
            stays.append((pt2 + subs[0][0], h, 0, ab2, anb2, pt2))
        cand = stays
        for h in hyps:
            ab, anb, pt, node, last, me, up, subs = h
            symbols = list(self.children[node])
            if node and self.spelled[node]:
                symbols.append(SEP)
            for v in symbols:
                if (me, v) in merged:
                    continue
                a = (ab if v == last else pt) + d[v] + (GAMMA if v == SEP else BETA)
                if a != -math.inf:
                    cand.append((a + subs[0][0], h, v, -math.inf, a, a))
        cut = max(x[0] for x in cand) - THETA
        cand = sorted((x for x in cand if x[0] >= cut), key=lambda x: -x[0])[:c.beam]
        out = []
        for _, h, v, ab, anb, pt in cand:
            if not v:
                out.append([ab, anb, pt] + h[3:])
                continue
            me = ids.setdefault((h[5], v), len(ids) + 1)
            if v == SEP:
                out.append([ab, anb, pt, 0, v, me, h[5], self.completed(h[7], self.spelled[h[3]])])
            else:
                out.append([ab, anb, pt, self.children[h[3]][v], v, me, h[5], h[7]])
        return out

    def output(self, hyps, end, words, scores):
        if end:
            self.fuse(hyps, True)
            whole = [h for h in hyps if h[3] == 0]
            hyps = whole or hyps
        for r, h in enumerate(sorted(hyps, key=lambda h: -(h[2] + h[7][0][0]))):
            scores[r] = h[2] + h[7][0][0]
            row = list(h[7][0][1][0])
            if end and self.c.marks:
                marks = marks_of(self.c, self.lm)
                row.append(max(marks, key=lambda m: self.bigram(row[-1] if row else self.lm.bos, m)))
            words[r, :len(row)] = row[:self.c.width]

    def decode(self, x, length, words, scores):
        c = self.c
        x = x.astype(np.float64)
        if c.raw:
            x = x - x.max(1, keepdims=True)
            x = x - np.log(np.exp(x).sum(1, keepdims=True))
        d, ids = ALPHA * x, {}
        hyps = [[0.0, -math.inf, 0.0, 0, 0, 0, -1, [(0.0, ((), (self.lm.bos, -1, -1), 0.0))]]]
        step = c.chunk or c.frames
        for k, lo in enumerate(range(0, c.frames, step)):
            for t in range(lo, min(lo + step, length)):
                hyps = self.frame(hyps, d[t].tolist(), ids)
                if c.interval and t and t % c.interval == 0:
                    self.fuse(hyps, False)
            self.output([list(h) for h in hyps], lo + step >= c.frames, words[k], scores[k])


def exact(case, seed):
    c = full(case)
    slow = 20 if c.words > 50_000 else 1  # sets of hundreds of homophones
    if c.batch * c.frames * c.beam * (1 + slow / 4) > 700_000:
        return None
    x, lengths, fusion_seed = inputs(c, seed)
    x, plain = x.cpu().numpy(), Plain(c, fusion_seed)
    calls = -(-c.frames // (c.chunk or c.frames))
    hyps = np.full((calls, c.batch, c.beam, c.width), -1, np.int32)
    scores = np.full((calls, c.batch, c.beam), -np.inf)
    for b in range(c.batch):
        plain.decode(x[b], int(lengths[b]), hyps[:, b], scores[:, b])
    return {"hyps": hyps, "scores": scores}
