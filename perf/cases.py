"""What the decoder is measured on: decoding as its users run it, from one short utterance on a
lexicon graph to several batches of 256 in flight on a 10 M state graph, offline, streaming and with
lattices.  Graphs, lengths, log-likelihood statistics and pruning follow workloads/configs.py.

The graph and the decoder handle are what a program creates once and keeps; they are kept here per
configuration too (a few at a time).  Log-likelihoods, utterance order and boosting targets come
from the seed."""
from __future__ import annotations

import math
from collections import OrderedDict

import numpy as np
import torch

from paper_2311_04996_amd import Decoder
from workloads import CONFIGS
from workloads.boost import boost_fsts
from workloads.configs import boost_tables, make_graph

# graph of a case -> configuration it is taken from
GRAPHS = {"lexicon": "c1_tiny", "medium": "c2_medium", "mini": "c3_mini", "large": "c3_large", "branchy": "c3_branchy"}
WORDS = {"lexicon": 200, "medium": 20_000, "mini": 200_000, "large": 200_000, "branchy": 200_000}
CLASSES = {"lexicon": 29, "medium": 129, "mini": 129, "large": 129, "branchy": 129}
ELEM = {"float32": 4, "float16": 2, "bfloat16": 2}

OFFLINE = dict(kind="offline", lo=50, hi=875, beam=17.0, max_active=10000, dtype="float32", boost="none",
               batches=1, host=False)
STREAM = dict(kind="stream", chunk=16, chunks=8, beam=17.0, max_active=10000, dtype="float32", boost="none")
LATTICE = dict(kind="lattice", lo=50, hi=300, beam=17.0, max_active=5000, dtype="float32", lattice_beam=4.0)


def listed():
    return [
        # a voice command against a small lexicon: the smallest call, 4 s of audio
        dict(OFFLINE, name="command", graph="lexicon", batch=1, lo=100, hi=100, beam=10.0, max_active=1000, host=True),
        # one dictated sentence of 12 s with the full language model: nothing else on the GPU
        dict(OFFLINE, name="one utterance", graph="large", batch=1, lo=300, hi=300, host=True),
        # transcribing a folder of recordings with a medium graph, 2 to 35 s each
        dict(OFFLINE, name="batch of 32", graph="medium", batch=32, max_active=7000),
        # the same with a list of 100 words to prefer per recording (names, products)
        dict(OFFLINE, name="batch of 32, word list", graph="medium", batch=32, hi=437, max_active=7000, boost="words"),
        # ... and with phrases of up to four words
        dict(OFFLINE, name="batch of 33, phrases", graph="medium", batch=33, hi=437, max_active=7000, boost="phrases"),
        # the throughput configuration: 256 recordings in one call
        dict(OFFLINE, name="batch of 256", graph="large", batch=256),
        # ... and as a transcription service runs it, several such batches in flight on batch slots
        dict(OFFLINE, name="6 batches in flight", graph="large", batch=256, batches=6),
        # fast first pass: tight pruning, half-precision scores from the acoustic model
        dict(OFFLINE, name="batch of 128, tight", graph="large", batch=128, beam=13.0, max_active=4000, dtype="float16"),
        # a graph in which every state branches (no state with the blank self-loop alone), bf16 scores
        dict(OFFLINE, name="batch of 64, branchy", graph="branchy", batch=64, hi=437, dtype="bfloat16"),
        # live captions for one speaker: 640 ms of audio at a time, a transcript after every chunk
        dict(STREAM, name="one stream", graph="large", channels=1),
        # a call centre: many streams advanced together, a transcript of each after every chunk
        dict(STREAM, name="512 streams", graph="large", channels=512, chunks=6),
        # lattices for rescoring: decode a few recordings and fetch every alternative near the best
        dict(LATTICE, name="lattices of 8", graph="large", batch=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: any graph, batch or stream count, length, pruning and input type."""
    kind = rng.choice(["offline", "offline", "offline", "stream", "stream", "lattice"])
    graph = rng.choice(["lexicon", "medium", "mini", "large", "large"])
    prune = dict(graph=graph, beam=round(rng.uniform(10.0, 17.0), 2), max_active=_log(rng, 1000, 10000),
                 dtype=rng.choice(["float32", "float32", "float16", "bfloat16"]))
    # (a phrase acceptor's states need room beside the graph's in a token's key: not on the larger graphs)
    boosts = ["none", "none", "none", "words"] + (["phrases"] if graph in ("lexicon", "medium") else [])
    if kind == "stream":
        chunk = _log(rng, 4, 32)
        return dict(STREAM, channels=_log(rng, 1, 512), chunk=chunk, chunks=rng.randint(2, max(2, min(10, 160 // chunk))),
                    boost=rng.choice(boosts), **prune)
    hi = _log(rng, 50, 875 if kind == "offline" else 400)
    batch = _log(rng, 1, 256 if kind == "offline" else 12)
    span = dict(batch=batch, lo=rng.randint(max(1, hi // 8), hi) if batch > 1 else hi, hi=hi)
    if kind == "lattice":
        prune["max_active"] = min(prune["max_active"], 6000)
        return dict(LATTICE, lattice_beam=round(rng.uniform(1.0, 6.0), 2), **span, **prune)
    batches = rng.randint(2, 3) if batch >= 32 and rng.random() < 0.3 else 1
    return dict(OFFLINE, boost=rng.choice(boosts), batches=batches, host=batches == 1 and rng.random() < 0.4,
                **span, **prune)


# ---- what a program keeps: graphs, decoders, streams
_graphs: dict = {}
_decoders: OrderedDict = OrderedDict()
_streams: list = []


def _graph(name):
    if name not in _graphs:
        _graphs[name] = make_graph(GRAPHS[name])
    return _graphs[name]


def _decoder(graph, workgroups=0, **options):
    key = (graph, workgroups, tuple(sorted(options.items())))
    if key not in _decoders:
        while len(_decoders) >= 4:
            _decoders.popitem(last=False)[1].close()
        _decoders[key] = Decoder(_graph(graph), **options)
        _decoders[key].set_launch_workgroups(workgroups)
    _decoders.move_to_end(key)
    return _decoders[key]


def _lengths(case, rng):
    """`batch` lengths evenly over lo..hi, in an order of the seed's."""
    n = np.round(np.linspace(case["lo"], case["hi"], case["batch"])).astype(np.int32)
    return rng.permutation(n)


def _loglikes(shape, seed, case):
    """Log-softmax rows as a CTC model gives them: the blank far ahead on most frames, on the others
    one token ahead."""
    ll = CONFIGS[GRAPHS[case["graph"]]]["ll"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = torch.empty(shape, dtype=getattr(torch, case["dtype"]), device="cuda")
    for b in range(0, shape[0], 64):                     # bounds the memory of the intermediate results
        part = (min(64, shape[0] - b),) + tuple(shape[1:])
        x = torch.randn(part, generator=gen, device="cuda") * ll["sigma"]
        blank = torch.rand(part[:-1], generator=gen, device="cuda") < ll["p_blank"]
        tok = torch.randint(1, part[-1], part[:-1], generator=gen, device="cuda")
        tok[blank] = 0
        up = torch.full(part[:-1], float(ll["token_boost"]), device="cuda")
        up[blank] = ll["blank_boost"]
        x.scatter_add_(-1, tok[..., None], up[..., None])
        out[b:b + part[0]] = torch.log_softmax(x, -1).to(out.dtype)
    return out


def _targets(case, n, seed):
    """Keyword arguments of decode_batch / init_channels: n streams' boosting targets."""
    if case["boost"] == "words":
        return dict(boosts=boost_tables(seed, n, WORDS[case["graph"]], min(100, WORDS[case["graph"]] // 4)))
    if case["boost"] == "phrases":
        return dict(boost_fsts=boost_fsts(seed, n, WORDS[case["graph"]], per_utt=100))
    return {}


def _out(n, words, host):
    if host:
        return (np.zeros((n, words), np.int32), np.zeros(n, np.int32), np.zeros(n, np.float32), np.zeros(n, np.int32))
    return tuple(torch.zeros(s, dtype=t, device="cuda") for s, t in
                 (((n, words), torch.int32), (n, torch.int32), (n, torch.float32), (n, torch.int32)))


def _transcripts(out):
    """Host results as a program reads them: the words that were found in every row, counts, costs, flags
    (what a row holds after its words is nobody's)."""
    words, n, cost, flags = out
    return [words * (np.arange(words.shape[1]) < n[:, None]), n, cost, flags]


def _hint(case):
    return max(4000, case["max_active"])                 # sizes the work buffers


# ---- the measured call
def prepare(case, seed):
    V = CLASSES[case["graph"]]
    rng = np.random.default_rng([seed, 0xCA5E])
    s = dict(case=case)
    if case["kind"] == "stream":
        n, C, K = case["channels"], case["chunk"], case["chunks"]
        # more streams than compute units: that many workgroups take the streams one after the other
        s["dec"] = _decoder(case["graph"], 256 if n > 256 else 0, max_channels=n, max_frames=C * K, max_words=128,
                            max_active_hint=_hint(case), outputs_on_host=True, loglike_dtype=case["dtype"])
        s["chunks"] = _loglikes((K, n, C, V), seed, case)
        s["channels"], s["frames"] = np.arange(n, dtype=np.int32), np.full(n, C, np.int32)
        s["targets"] = _targets(case, n, seed)
        s["out"] = [_out(n, 128, True) for _ in range(K)]
        return s
    B, k = case["batch"], case.get("batches", 1)
    lattice = case["kind"] == "lattice"
    # arenas for the mean utterance (lattice_by_length shares them out)
    mean = (case["lo"] + case["hi"]) / 2 + 2
    slots = min(3, k)
    options = dict(max_channels=B * slots, max_frames=case["hi"], max_words=256, max_active_hint=_hint(case),
                   outputs_on_host=case.get("host", False), loglike_dtype=case["dtype"])
    if lattice:
        options.update(keep_token_records=True)
    else:
        options.update(batch_slots=slots, lattice_by_length=True,
                       lattice_bytes_per_channel=int(8 * 1.5 * _hint(case) * (mean + 1)))
    # several batches in flight: half of the 256 compute units to each launch
    s["dec"] = _decoder(case["graph"], 128 if k > 1 else 0, **options)
    s["lengths"] = [_lengths(case, rng) for _ in range(k)]
    s["ll"] = [_loglikes((B, case["hi"], V), seed * 16 + i, case) for i in range(k)]
    if lattice:
        s["out"] = [_out(B, 256, False)]
        cells = int(sum(s["lengths"][0]) + B) * 2 * _hint(case)      # room for every token's or link's cost
        s["costs"] = [torch.zeros(cells, device="cuda"), torch.zeros(2 * cells, device="cuda")]
        return s
    s["targets"] = [_targets(case, B, seed * 16 + i) for i in range(k)]
    s["out"] = [_out(B, 256, case["host"]) for _ in range(k)]
    if k > 1:
        while len(_streams) < 3:
            _streams.append(torch.cuda.Stream())
    return s


def run(s):
    case, dec = s["case"], s["dec"]
    beam, max_active = case["beam"], case["max_active"]
    if case["kind"] == "stream":
        last, got = len(s["out"]) - 1, []
        dec.init_channels(s["channels"], beam, max_active, **s["targets"])
        for k, out in enumerate(s["out"]):
            dec.advance_chunk_partial(s["channels"], s["chunks"][k], s["frames"], finalize=k == last, out=out)
            got.append(_transcripts(out))
        return got
    if case["kind"] == "lattice":
        out = dec.decode_batch(s["ll"][0], s["lengths"][0], beam, max_active, out=s["out"][0])
        chans = np.arange(case["batch"], dtype=np.int32)
        off, tok_first, link_first, _, cost, links = dec.get_lattice_batch(chans, s["ll"][0], s["lengths"][0],
                                                                           case["lattice_beam"], on_device=True)
        # a set's tokens and links come in no particular order: all token costs and all link costs, sorted
        for all_costs, c in zip(s["costs"], (cost, links.view(torch.float32).view(-1, 8)[:, 6])):
            all_costs[:c.numel()] = torch.sort(c)[0]
        return [out, off, tok_first, link_first, *s["costs"]]
    k = len(s["out"])
    if k == 1:
        dec.decode_batch(s["ll"][0], s["lengths"][0], beam, max_active, out=s["out"][0], **s["targets"][0])
    else:
        now = torch.cuda.current_stream()
        for i in range(k):
            st = _streams[i % 3]
            st.wait_stream(now)
            dec.decode_batch(s["ll"][i], s["lengths"][i], beam, max_active, out=s["out"][i], slot=i % 3, stream=st,
                             **s["targets"][i])
        for st in _streams:
            now.wait_stream(st)
    return [_transcripts(o) for o in s["out"]] if case["host"] else s["out"]


# ---- what a pass cannot do without
def _tokens_per_frame(case):
    """Tokens of a closed set, from the decoder's counters over these graphs (an average; it depends
    on the scores): what the beam lets through, at most about max-active."""
    if case["graph"] == "lexicon":
        return min(1750.0, 0.95 * case["max_active"])
    if case["graph"] == "medium":
        return 1.16 * case["max_active"]
    by_beam = 1732.0 * math.exp(0.465 * (case["beam"] - 10.0))
    return min(by_beam, 1.03 * case["max_active"] ** 1.3 / 10000 ** 0.3)


def work(case):
    """Per frame a row of scores; per token its record and its state's (24 bytes), its arcs (2.3
    emitting of 12 bytes, 0.5 epsilon of 8) and, once it is a survivor, a candidate, a queue record and
    a backpointer (32); two additions per arc."""
    if case["kind"] == "stream":
        frames = case["channels"] * case["chunk"] * case["chunks"]
    else:
        frames = case["batch"] * (case["lo"] + case["hi"]) / 2 * case.get("batches", 1)
    tokens = _tokens_per_frame(case)
    n = {"bytes": frames * (CLASSES[case["graph"]] * ELEM[case["dtype"]] + 88.0 * tokens), "flops": frames * tokens * 5.6}
    if case["kind"] == "lattice":                        # tokens read again and written, 1.3 links of 32 bytes each
        n["bytes"] += frames * tokens * (16 + 8 + 1.3 * 32)
    return n


def tolerance(case):
    # costs are sums in one fixed order in fp32 and ties have a rule: every implementation gets these bits
    return "exact"
