"""The constants of the built-in kernel choice (kCost24, kCostDense and kCost48 in matmul.hip) from the times in
kernel_choice_times.csv: a least-squares fit of the relative error per kernel, no constant negative.  Prints for every pattern
the largest difference from the constants in the source, and how the choice made with them compares with the fastest kernel and
with the rule it replaced.  The same for the row of the pairs kernel (kernel_choice_pairs_times.csv) and for the decode kernels that keep the
tokens' rows (kFold24, kFoldDense and kFold48, from kernel_choice_rows_times.csv), whose calls through the built-in choice
kernel_choice_rows_calls.csv compares with those before.

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
ROWS_TABLES = {"2:4": "kFold24", "dense": "kFoldDense", "4:8": "kFold48"}
PAIRS, PAIRS_FACTOR = "pairs_w8_r128_t64", 1.2  # its row stands that much higher than its fit
STREAM = {8: "stream_w8_r1_d3", 9: "stream_w9_r1_d3", 11: "stream_w11_r1_d3"}


def ceil_div(a, b):
    return -(-a // b)


def read_csv(name):
    return list(csv.reader(l for l in open(os.path.join(HERE, name)) if not l.startswith("#")))


def read_times(name, first):
    """Per pattern (M, N, K, the columns up to `first`, {kernel: time}); a file may have a heading for each pattern."""
    rows = {p: [] for p in TABLES}
    for line in read_csv(name):
        if line[0] == "pattern":
            names = line[first:]
            continue
        M, N, K = map(int, line[1:4])
        rows[line[0]].append((M, N, K, *map(float, line[4:first]), {n: float(t) for n, t in zip(names, line[first:]) if t}))
    return rows


def read_source():
    text = open(SOURCE).read()
    variants = {}
    for name, kind, rest in re.findall(r'\{"(\w+)", KIND_(\w+), ([^}]*)\}', text):
        f = [int(x) for x in rest.split(",")] + [0] * 9
        variants[name] = dict(kind=kind, rt=f[0], tt=f[1], split=f[2], nw=f[3], half=f[7])
    tables = {}
    for table in [*TABLES.values(), *ROWS_TABLES.values()]:
        body = text[text.index(table + "[] = {"):]
        body = body[:body.index("};")]
        tables[table] = {n: np.array([float(x.strip()[:-1]) for x in c.split(",")])
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


def apart(again, constants, data):
    """Largest difference of a term of the estimate, as a share of the time, at the middle of the data."""
    typical = np.median([d[0] for d in data], axis=0)
    return float(np.abs((again - constants) * typical).max() / np.median([d[1] for d in data]))


def geo(v):
    return math.exp(np.mean(np.log(v)))


def single_products(variants, tables):
    for pattern, rows in read_times("kernel_choice_times.csv", 5).items():
        table = {n: c for n, c in tables[TABLES[pattern]].items() if n != PAIRS}
        usable = lambda n, M: not (n.startswith("ksplit") and M > 64)  # 4:8: 64 tokens at a time
        off = 0.0
        for name, constants in table.items():
            shared = name.startswith("stream")  # one fit for the three, each where it is the one that would run
            data = [(quantities(variants[n], pattern, M, N, K), t[n]) for M, N, K, _, t in rows
                    for n in ([aligned_stream(N, K)] if shared else [name]) if n in t and usable(n, M)]
            off = max(off, apart(fit([d[0] for d in data], [d[1] for d in data]), constants, data))
        chosen, rule, slower = [], [], []
        for M, N, K, old, t in rows:
            can = [n for n in t if n in table and usable(n, M) and (not n.startswith("stream") or n == aligned_stream(N, K))]
            pick = min(can, key=lambda n: float(np.dot(quantities(variants[n], pattern, M, N, K), table[n])))
            best = min(min(t.values()), old)
            chosen.append(t[pick] / best)
            rule.append(old / best)
            if t[pick] > 1.03 * old:
                slower.append((t[pick] / old, M, N, K, pick))
        print("%-5s %d products, %d weight shapes; refit within %.2f %% of a time; chosen / fastest: mean %.3f, worst %.2f; rule / fastest: "
              "mean %.3f, worst %.2f; over 3 %% slower than the rule: %d" % (pattern, len(rows), len({r[1:3] for r in rows}), 100 * off,
                                                                          geo(chosen), max(chosen), geo(rule), max(rule), len(slower)))
        for s in sorted(slower, reverse=True):
            print("      %.3f x the rule's time: %d x %d x %d %s" % s)


def pairs_kernel(variants, tables):
    table = tables[TABLES["2:4"]]
    lines = [(*map(int, l[:3]), *map(float, l[3:])) for l in read_csv("kernel_choice_pairs_times.csv")[1:]]
    one = [l for l in lines if ceil_div(l[1], 128) * ceil_div(l[0], 64) <= 256]  # one macro tile per CU at most
    data = [(quantities(variants[PAIRS], "2:4", *l[:3]), l[3]) for l in one]
    keep = [0, 1, 3]  # launch, steps, memory: with one round the other terms say the same
    again = np.zeros(7)
    again[keep] = fit([[d[0][i] for i in keep] for d in data], [d[1] for d in data])
    error = np.mean([abs(np.dot(d[0], again) / d[1] - 1) for d in data])
    for factor in (1.0, PAIRS_FACTOR):
        ratio = []
        for M, N, K, pairs, choice in one:
            can = [n for n in table if n != PAIRS and not n.startswith("ksplit") and (not n.startswith("stream") or (M <= 128 and n == aligned_stream(N, K)))
                   and not (variants[n]["split"] and variants[n]["kind"] == "TILE" and M > 512)]
            others = min(float(np.dot(quantities(variants[n], "2:4", M, N, K), table[n])) for n in can)
            ratio.append(pairs / choice if factor * np.dot(quantities(variants[PAIRS], "2:4", M, N, K), again) < others else 1.0)
        print("pairs %d products, %d of at most 256 macro tiles, mean error %.3f; row %.2f x the fit: refit within %.2f %% of a time; taken for %d, call / "
              "without: mean %.3f, worst %.2f, over 1.06: %d" % (len(lines), len(one), error, factor, 100 * apart(PAIRS_FACTOR * again, table[PAIRS], data),
                                                              sum(r != 1.0 for r in ratio), geo(ratio), max(ratio), sum(r > 1.06 for r in ratio)))


def rows_quantities(v, pattern, M, N, K):
    """As quantities, of a decode kernel that keeps the tokens' rows: `tokens` are the bytes of rows and places that a CU copies."""
    q = quantities(v, pattern, M, N, K)
    per = ceil_div(ceil_div(ceil_div(N, 16), v["rt"]), 256)
    q[2] = per * ((2 if M > 8 else 1) * (K + 8) * 16 + ceil_div(K, 256) * 512)
    return q


def rows_fitted(name, v, M, N, K):
    """The calls of the fit: around those that the rule on waves, row tiles, workgroups per CU and bytes lets in."""
    per, kb = ceil_div(ceil_div(ceil_div(N, 16), v["rt"]), 256), ((2 if M > 8 else 1) * (K + 8) * 16 + ceil_div(K, 256) * 512) / 1024
    if max(kb, v["nw"] * v["rt"]) > 158:
        return False
    quads = name.endswith("_q")
    if v["nw"] == 16:
        return per == 1 or per * kb <= 160 or (kb <= 40 and per <= 4)
    if kb <= 40:
        return per <= 4 and not (v["rt"] == 4 and quads)
    if kb <= 76:
        return v["rt"] >= 2 if per == 2 else per == 1 and (v["rt"] <= 2 or v["rt"] == 6)
    return per == 1 and (v["rt"] == 6 or (v["rt"] == 2 and kb <= 96) or (v["rt"] == 1 and quads))


def rows_kept(variants, tables):
    calls = read_csv("kernel_choice_rows_calls.csv")[1:]
    for pattern, rows in read_times("kernel_choice_rows_times.csv", 4).items():
        off, errors = 0.0, []
        for name, constants in tables[ROWS_TABLES[pattern]].items():
            data = [(rows_quantities(variants[name], pattern, M, N, K), t[name]) for M, N, K, t in rows if name in t and rows_fitted(name, variants[name], M, N, K)]
            again = fit([d[0] for d in data], [d[1] for d in data])
            off = max(off, apart(again, constants, data))
            errors += [abs(np.dot(d[0], again) / d[1] - 1) for d in data]
        ratio = [float(l[5]) / min(float(l[4]), float(l[6])) for l in calls if l[0] == pattern]
        print("%-5s rows kept: %d calls of %d weight shapes, mean error %.3f; refit within %.2f %% of a time; %d calls, after / before: mean %.3f, worst %.3f"
              % (pattern, len(rows), len({r[1:3] for r in rows}), np.mean(errors), 100 * off, len(ratio), geo(ratio), max(ratio)))


def main():
    source = read_source()
    single_products(*source)
    pairs_kernel(*source)
    rows_kept(*source)


if __name__ == "__main__":
    main()
