"""The constants of the built-in kernel choice (kCost24, kCostDense and kCost48 in matmul.hip) from the times in
kernel_choice_times.csv: a least-squares fit of the relative error per kernel, no constant negative.  Prints for every pattern
the largest difference from the constants in the source, and how the choice made with them compares with the fastest kernel and
with the rule it replaced.

    python3 profiles/kernel_choice_fit.py
"""
import csv
import math
import os
import re

import numpy as np
from scipy.optimize import nnls

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "..", "paper_2310_15929_amd", "csrc", "matmul.hip")
TABLES = {"2:4": "kCost24", "dense": "kCostDense", "4:8": "kCost48"}
STREAM = {8: "stream_w8_r1_d3", 9: "stream_w9_r1_d3", 11: "stream_w11_r1_d3"}


def ceil_div(a, b):
    return -(-a // b)


def read_times():
    rows, names = {p: [] for p in TABLES}, None
    for line in csv.reader(l for l in open(os.path.join(HERE, "kernel_choice_times.csv")) if not l.startswith("#")):
        if line[0] == "pattern":
            names = line[5:]
            continue
        M, N, K = map(int, line[1:4])
        rows[line[0]].append((M, N, K, float(line[4]), {n: float(t) for n, t in zip(names, line[5:]) if t}))
    return rows


def read_source():
    text = open(SOURCE).read()
    variants = {}
    for name, kind, rest in re.findall(r'\{"(\w+)", KIND_(\w+), ([^}]*)\}', text):
        f = [int(x) for x in rest.split(",")] + [0] * 9
        variants[name] = dict(kind=kind, rt=f[0], tt=f[1], split=f[2], nw=f[3], half=f[7])
    tables = {}
    for pattern, table in TABLES.items():
        body = text[text.index(table + "[] = {"):]
        body = body[:body.index("};")]
        tables[pattern] = {n: np.array([float(x.strip()[:-1]) for x in c.split(",")])
                           for n, c in re.findall(r'\{"(\w+)", ([^}]*)\}', body)}
    return variants, tables


def stream_span(nrb, nks):
    span = max(ceil_div(nrb * nks, 256), 8, ceil_div(nks, 14))
    span = ceil_div(span, 2) * 2
    for a in range(span, nks + 1, 2):
        if a * 5 > span * 6:
            break
        if nks % a == 0:
            return a
    return span


def aligned_stream(N, K):
    nrt, nks = ceil_div(N, 16), ceil_div(K, 256) * 4
    best, pick = 0, 8
    for nw in STREAM:
        nrb = ceil_div(nrt, nw)
        if nrb > 256:
            continue
        p = 256 // nrb
        while p > 1 and (nks % p or (nks // p) % 2 or nks // p < 8):
            p -= 1
        if nrb * p > best:
            best, pick = nrb * p, nw
    return STREAM[pick if best >= 200 else 8]


def quantities(v, pattern, M, N, K):
    """What the seven constants multiply: 1, weights, tokens, memory, partial, reduce, rounds."""
    nrt, nks, Mt = ceil_div(N, 16), ceil_div(K, 256) * 4, ceil_div(M, 16)
    wb = 2.0 if pattern == "dense" else 1.125
    memory, out, pieces = nrt * 16 * nks * 64 * wb, 8.0 * M * nrt * 16, 0.0
    if v["kind"] == "KSPLIT":
        ns = v["tt"] if v["split"] else 1
        per = ceil_div(ceil_div(nrt, v["rt"]) * ns, 256)
        token_bytes = 2 * (1 << (M - 1).bit_length()) if M <= 16 else 32 * (2 if M <= 32 else 4)
        weights, tokens, rounds = per * nks / ns * 64 * 16 * wb * v["rt"], per * nks / ns * 64 * token_bytes, per
        pieces = ns if ns > 1 else 0.0
    elif v["kind"] == "STREAM":
        rows = v["nw"] * v["rt"]
        nrb = ceil_div(nrt, rows)
        span = stream_span(nrb, nks)
        mt = 1 if Mt <= 1 else 2 if Mt <= 2 else 4 if Mt <= 4 else 8
        weights, tokens, rounds = span * 64 * 16 * wb * rows, span * 64 * 32 * mt, span
        pieces = max(1.0, ceil_div(nrb * nks, span) / nrb) if span % nks else 0.0
    else:
        rows = 2 * v["rt"] if pattern != "dense" or v["half"] else 2 * (v["rt"] // 2)
        h = 2 if v["half"] else 1
        tiles, ns, st = ceil_div(nrt, rows) * ceil_div(Mt, v["nw"] * v["tt"]), 1, nks * h
        if v["split"]:
            room = 16 if M <= 128 else (4 if M <= 512 else 1)
            want = 256 // tiles if M > 128 else (1 if tiles >= 128 else ceil_div(512, tiles))
            ns = max(1, min(want, st // 8, room))
            st = ceil_div(ceil_div(st, ns), 4) * 4
            ns = ceil_div(nks * h, st)
        per = ceil_div(tiles * ns, 256)
        weights, tokens, rounds = per * st / h, per, max(1.0, tiles * ns / 256) * st / h
        pieces = ns if ns > 1 else 0.0
    return [1.0, weights, tokens, memory, out * pieces, 1.0 if pieces else 0.0, rounds]


def fit(x, y):
    x, y = np.array(x), np.array(y)
    scale = x.max(axis=0)
    scale[scale == 0] = 1
    return nnls(x / scale / y[:, None], np.ones(len(y)))[0] / scale


def main():
    variants, tables = read_source()
    for pattern, rows in read_times().items():
        table = tables[pattern]
        usable = lambda n, M: not (n.startswith("ksplit") and M > 64)  # 4:8: 64 tokens at a time
        off = 0.0
        for name, constants in table.items():
            shared = name.startswith("stream")  # one fit for the three, each where it is the one that would run
            data = [(quantities(variants[n], pattern, M, N, K), t[n]) for M, N, K, _, t in rows
                    for n in ([aligned_stream(N, K)] if shared else [name]) if n in t and usable(n, M)]
            again = fit([d[0] for d in data], [d[1] for d in data])
            typical = np.median([d[0] for d in data], axis=0)
            off = max(off, float(np.abs((again - constants) * typical).max() / np.median([d[1] for d in data])))
        chosen, rule, slower = [], [], []
        for M, N, K, old, t in rows:
            can = [n for n in t if n in table and usable(n, M) and (not n.startswith("stream") or n == aligned_stream(N, K))]
            pick = min(can, key=lambda n: float(np.dot(quantities(variants[n], pattern, M, N, K), table[n])))
            best = min(min(t.values()), old)
            chosen.append(t[pick] / best)
            rule.append(old / best)
            if t[pick] > 1.03 * old:
                slower.append((t[pick] / old, M, N, K, pick))
        geo = lambda v: math.exp(np.mean(np.log(v)))
        print("%-5s %d products, %d weight shapes; refit within %.2f %% of a time; chosen / fastest: mean %.3f, worst %.2f; rule / fastest: "
              "mean %.3f, worst %.2f; over 3 %% slower than the rule: %d" % (pattern, len(rows), len({r[1:3] for r in rows}), 100 * off,
                                                                          geo(chosen), max(chosen), geo(rule), max(rule), len(slower)))
        for s in sorted(slower, reverse=True):
            print("      %.3f x the rule's time: %d x %d x %d %s" % s)


if __name__ == "__main__":
    main()
