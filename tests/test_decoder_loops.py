"""The decoder's whole time loop in one launch (csrc/loop.hip), forward and backward, against the launch per layer and position
(CMT_DEC_LOOP=0, read when the handle is created) and against the oracle; the plan of its workgroups on the CPU."""
import os
import subprocess
import threading

import numpy as np
import pytest

from oracle import nmt_oracle as O
from paper_1802_07170_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "paper_1802_07170_amd/csrc/recur_plan.h"
int main() {
  using namespace cmt;
  for (int prec = 0; prec < 2; ++prec)
    for (int H = 16; H <= 1024; H += 16)
      for (int Bp = 16; Bp <= 256; Bp += 16)
        for (int L = 1; L <= 8; ++L)
          for (int cus = 64; cus <= 256; cus += 64) {
            const LoopPlan p = loop_plan(prec, L, Bp, H, 60, cus);
            const bool wanted = L <= 4 && Bp <= 128 && H / 4 <= cus && (prec || H <= 512) && cus == 256;
            if (!p.ok) {
              if (wanted) { printf("%d %d %d %d %d: refused\n", prec, H, Bp, L, cus); return 1; }
              continue;
            }
            // every workgroup on the chip at once, every sentence in a group, no empty group, chunks that hold a group's tiles,
            // 8 wavefronts of nk steps that cover the width
            const bool ok = p.groups * p.nwg <= cus && p.groups * p.tiles * 16 >= Bp && (p.groups - 1) * p.tiles * 16 < Bp && p.tiles <= 8 &&
                            p.bt * p.nch >= p.tiles && 8 * p.nk * 32 >= H && p.nwg * 4 == H && L <= 4;
            if (!ok) { printf("%d %d %d %d %d\n", prec, H, Bp, L, cus); return 1; }
          }
  return 0;
}
"""


def _compile_and_run(tmp_path, program, *args):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{ROOT}", str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True)


def test_every_workgroup_of_a_loop_fits_the_chip(tmp_path):
    r = _compile_and_run(tmp_path, PROGRAM)
    assert r.returncode == 0, r.stdout


PAYS = r"""
#include <stdio.h>
#include <stdlib.h>
#include "paper_1802_07170_amd/csrc/recur_plan.h"
int main(int argc, char** argv) {
  using namespace cmt;
  for (int i = 1; i + 5 < argc; i += 6) {
    int v[6];
    for (int k = 0; k < 6; ++k) v[k] = atoi(argv[i + k]);
    const LoopPlan p = loop_plan(v[0], v[2], (v[3] + 15) / 16 * 16, v[1], v[4], 256);
    putchar('0' + (p.ok && (v[5] > 0 ? loop_pays(p, v[2], v[5]) : loop_decode_pays(p, v[0], v[2], v[1], -v[5]))));
  }
  return 0;
}
"""


def test_loops_are_taken_where_they_are_faster(tmp_path):
    """Shapes measured on both sides of the lines by 7 % and more (precision, hidden, layers, sentences, source length, target
    length, or for a translation minus the vocabulary), and the usual ones."""
    faster = [(1, 16, 1, 16, 24, 40), (1, 32, 1, 128, 128, 40), (1, 48, 3, 16, 128, 40), (0, 16, 2, 128, 64, 40), (1, 64, 1, 16, 20, 3), (1, 64, 1, 8, 10, 10),
              (1, 1024, 4, 64, 50, 50), (0, 512, 2, 64, 50, 50), (1, 512, 2, 32, 120, 120), (1, 1024, 4, 128, 80, 80), (1, 1024, 4, 64, 50, -32000),
              (0, 512, 2, 1, 25, -32000), (1, 16, 1, 16, 20, -768), (0, 128, 4, 16, 20, -9216), (1, 512, 1, 64, 20, -49152), (0, 256, 1, 16, 20, -24576)]
    slower = [(1, 16, 1, 16, 64, 40), (0, 16, 1, 16, 128, 40), (1, 32, 1, 16, 128, 40), (1, 16, 2, 16, 96, 40), (1, 512, 2, 16, 20, 1), (1, 16, 1, 16, 20, -1536),
              (0, 64, 1, 16, 20, -6144), (0, 128, 2, 16, 20, -12288), (1, 16, 2, 16, 100, -768), (1, 64, 2, 16, 100, -6144), (1, 256, 1, 16, 20, -24576)]
    r = _compile_and_run(tmp_path, PAYS, *(x for c in faster + slower for x in c))
    assert r.stdout == "1" * len(faster) + "0" * len(slower)


# How the passes of a handle ran, by (CMT_DEC_LOOP, CMT_RECUR): a training step has two loops, an evaluation or a translation one.
# Without this the comparisons below could not tell: a loop that gave up all its waits is made again by the form without
# any, and one that was refused runs as the launches that it is compared with.
def _ran_as_asked(tr, loops, again):
    got_loops, got_again = tr.wait_counts()
    assert got_loops == loops, (got_loops, loops)
    assert (got_again > 0) == again, got_again


def _step(cfg, batch, B, S, T, prec, reg=None, steps=1, loops=True, give_up=False):
    """Losses and gradients of a step and the evaluation after it, and that the decoder's loops were taken or not, and their waits
    given up or not, as the caller expects."""
    from paper_1802_07170_amd import binding
    tr = binding.Trainer(cfg, B, S, T, precision=prec)
    tr.set_params(I.flatten(I.make_params(cfg, 11, 0.05), cfg))
    dev = tr.upload_batch(*batch)
    if reg:
        tr.set_regularization(*reg)
    for _ in range(steps):
        loss = tr.train_step(dev)
    grads = tr.get_grads()
    eval_loss = tr.eval_loss(dev)
    _ran_as_asked(tr, 2 * steps + 1 if loops else 0, give_up)
    tr.close()
    return loss, grads, eval_loss


def _batch(cfg, B, S, T, seed):
    rng = np.random.default_rng(seed)
    src_len, tgt_len = rng.integers(1, S + 1, B).astype(np.int32), rng.integers(1, T + 1, B).astype(np.int32)
    src_len[rng.integers(B)], tgt_len[rng.integers(B)] = S, T
    src = rng.integers(4, cfg["src_vocab"], (B, S)).astype(np.int32)
    tgt = rng.integers(4, cfg["tgt_vocab"], (B, T)).astype(np.int32)
    src[np.arange(S) >= src_len[:, None]] = 0
    tgt[np.arange(T) >= tgt_len[:, None]] = 0
    return src, src_len, tgt, tgt_len


# one, two, three, four, five and eight tiles of sentences per group, one to four layers, widths that end in half a k step or in the
# middle of a wavefront's steps, one position, source lengths at the edges of the mix's shares (8 and 16 per thread)
SHAPES = [(1, 1, 1, 16, 8, 1), (17, 3, 2, 48, 24, 2), (5, 128, 3, 64, 64, 1), (40, 9, 5, 336, 40, 3), (64, 65, 4, 256, 32, 4),
          (70, 64, 3, 528, 16, 1), (33, 20, 4, 512, 64, 2), (128, 33, 3, 512, 16, 2), (112, 12, 2, 272, 16, 2)]
WIDE = [(20, 7, 3, 1024, 64, 4), (64, 70, 3, 784, 32, 4), (80, 65, 2, 1024, 64, 2), (128, 17, 3, 1024, 64, 3)]


@pytest.mark.gpu
@pytest.mark.parametrize("reg", [None, (0.3, 0.1, 5)], ids=["plain", "dropout"])
@pytest.mark.parametrize("prec,B,S,T,H,E,L", [(0, *s) for s in SHAPES if s[3] <= 512] + [(1, *s) for s in SHAPES + WIDE])
def test_loops_agree_with_the_launch_per_position(prec, B, S, T, H, E, L, reg, monkeypatch):
    """Both forms take the same operands at the same precision and add the same products in another order.  fp32: the parity
    bar of 1e-4 holds between either form and the oracle, the forms differ by far less.  16-bit operands: a rounding of a
    state or gate gradient that falls the other way is 2^-9 of it, and the two forms' gradients differ by a few parts in
    10^3 (the attention's own matrix by more: its gradient is what is left after the softmax Jacobian has cancelled the rest)."""
    cfg = dict(src_vocab=128, tgt_vocab=136, emb=E, hidden=H, layers=L)
    batch = _batch(cfg, B, S, T, seed=H + B)
    res = {}
    for mode, switch in (("0", "0"), ("1", "2")):         # (2: also where launches would be faster)
        monkeypatch.setenv("CMT_DEC_LOOP", switch)
        res[mode] = _step(cfg, batch, B, S, T, prec, reg, loops=mode == "1")
    assert abs(res["0"][0] - res["1"][0]) <= (1e-6 if prec == 0 else 2e-4) * abs(res["0"][0])
    assert abs(res["0"][2][0] - res["1"][2][0]) <= (1e-6 if prec == 0 else 2e-4) * abs(res["0"][2][0])
    a, b = I.unflatten(res["0"][1], cfg), I.unflatten(res["1"][1], cfg)
    bar = 1e-4 if prec == 0 else 2e-2
    total = np.linalg.norm(res["0"][1].astype(np.float64))
    for name in a:
        x, y = a[name].astype(np.float64), b[name].astype(np.float64)
        assert np.isfinite(y).all(), name
        diff, norm = np.linalg.norm(x - y), np.linalg.norm(x)
        if name == "W_a" or norm < 1e-4 * total:          # (nearly cancelled: held against the whole gradient)
            assert diff <= bar * 1e-2 * total, (name, diff, norm, total)
        else:
            assert diff <= bar * norm, (name, diff, norm)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,B,S,T,H,E,L", [(0, 20, 9, 6, 80, 24, 2), (1, 20, 9, 6, 96, 32, 3), (0, 7, 40, 3, 16, 8, 4), (1, 33, 12, 4, 144, 48, 1)])
@pytest.mark.parametrize("give_up", [False, True], ids=["together", "waits given up"])
def test_loops_match_the_oracle(prec, B, S, T, H, E, L, give_up, monkeypatch):
    """Also where every wait is given up at once (CMT_RECUR=2): the launch behind each loop then makes it again without waits."""
    cfg = dict(src_vocab=128, tgt_vocab=136, emb=E, hidden=H, layers=L)
    batch = _batch(cfg, B, S, T, seed=B)
    params = I.make_params(cfg, 11, 0.05)
    oloss, og, _ = O.train_step(cfg, params, *batch)
    if give_up:
        monkeypatch.setenv("CMT_RECUR", "2")
    loss, grads, _ = _step(cfg, batch, B, S, T, prec, steps=2, give_up=give_up)
    bar = 1e-4 if prec == 0 else 2e-2
    assert abs(loss - oloss) <= bar * abs(oloss)
    g = I.unflatten(grads, cfg)
    for name, want in og.items():
        if prec and name == "W_a":                        # (ill-conditioned: see the tests of the conditioning)
            continue
        assert np.linalg.norm(g[name] - want) <= bar * np.linalg.norm(want) + 1e-12, name


@pytest.mark.gpu
@pytest.mark.parametrize("prec,B,S,T,H,E,L", [(1, 24, 9, 6, 528, 32, 2), (1, 128, 70, 3, 64, 32, 4), (0, 24, 9, 6, 272, 32, 2)])
def test_loops_without_waits_give_the_same(prec, B, S, T, H, E, L, monkeypatch):
    """The form without waits at shapes and with dropout that the oracle test above does not reach; the bars as there."""
    cfg = dict(src_vocab=128, tgt_vocab=136, emb=E, hidden=H, layers=L)
    batch = _batch(cfg, B, S, T, seed=3)
    a = _step(cfg, batch, B, S, T, prec, (0.2, 0.1, 9))
    monkeypatch.setenv("CMT_RECUR", "2")
    b = _step(cfg, batch, B, S, T, prec, (0.2, 0.1, 9), give_up=True)
    assert abs(a[0] - b[0]) <= (1e-6 if prec == 0 else 2e-4) * abs(a[0])
    x, y = a[1].astype(np.float64), b[1].astype(np.float64)
    assert np.linalg.norm(x - y) <= (1e-5 if prec == 0 else 1e-2) * np.linalg.norm(x)


@pytest.mark.gpu
def test_loops_of_several_streams_and_threads():
    """Handles on their own streams, from their own threads: a loop takes the whole chip, and they take turns."""
    from paper_1802_07170_amd import binding
    import torch
    cfg = dict(src_vocab=128, tgt_vocab=136, emb=32, hidden=512, layers=2)
    batch = _batch(cfg, 32, 20, 12, seed=1)
    want = _step(cfg, batch, 32, 20, 12, 1, steps=1)[1]
    trainers = []
    for _ in range(3):
        with torch.cuda.stream(torch.cuda.Stream()):
            tr = binding.Trainer(cfg, 32, 20, 12, precision=1)
            tr.set_params(I.flatten(I.make_params(cfg, 11, 0.05), cfg))
            trainers.append((tr, tr.upload_batch(*batch)))
    torch.cuda.synchronize()
    got = [None] * len(trainers)

    def work(i):
        tr, dev = trainers[i]
        for _ in range(6):
            tr.train_step_async(dev)
        tr.fetch_loss()
        got[i] = tr.get_grads()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(trainers))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for g in got:
        np.testing.assert_array_equal(g, want)
    for tr, _ in trainers:
        _ran_as_asked(tr, 12, False)
        tr.close()


@pytest.mark.gpu
@pytest.mark.parametrize("prec,B,S,T,H,E,L,V", [(0, 1, 5, 7, 64, 40, 1, 1000), (0, 40, 9, 6, 336, 72, 3, 136), (0, 64, 20, 9, 256, 256, 2, 5000),
                                                (0, 128, 12, 5, 512, 16, 4, 2056), (1, 17, 9, 9, 48, 24, 2, 136), (1, 64, 30, 8, 1024, 1160, 4, 1016),
                                                (1, 3, 9, 8, 528, 2048, 2, 8008), (1, 100, 9, 8, 512, 512, 1, 2000), (0, 5, 9, 8, 16, 8, 1, 16000)])
@pytest.mark.parametrize("give_up", [False, True], ids=["together", "waits given up"])
def test_greedy_loop_gives_the_tokens_of_the_launches(prec, B, S, T, H, E, L, V, give_up, monkeypatch):
    """The whole search in one launch against a launch per layer and step (CMT_DEC_LOOP=0); the last shape's vocabulary is too long
    for its width and takes the launches both times.  Weights of twice a layer's usual scale make the tokens vary (27 - 572 different
    ones over these shapes); the end token is one that ends some sentences early.  In fp32 all tokens agree; with 16-bit operands a
    near tie may turn, and with it the rest of that sentence.  The two differ in the order of 32-bit sums and in the few 16-bit roundings
    that this turns, so fewer sentences may part than 16-bit operands make part from 32-bit ones, which most do not."""
    from paper_1802_07170_amd import binding
    cfg = dict(src_vocab=128, tgt_vocab=V, emb=E, hidden=H, layers=L)
    params = I.make_params(cfg, 11, 3.4 / np.sqrt(H))
    params["E_tgt"] *= np.sqrt(H) / 2
    params["E_src"] *= np.sqrt(H) / 2
    src, src_len, _, _ = _batch(cfg, B, S, T, seed=B)
    res, eos = {}, 3
    for mode in ("any end", "fp32", "0", "1"):
        monkeypatch.setenv("CMT_DEC_LOOP", "1" if mode == "1" else "0")
        if mode == "1" and give_up:
            monkeypatch.setenv("CMT_RECUR", "2")
        tr = binding.Trainer(cfg, B, S, T, precision=0 if mode == "fp32" else prec)
        tr.set_params(I.flatten(params, cfg))
        for _ in range(2):                                # (the second time on the memory that the first left behind)
            ids, lens = tr.greedy_decode(src, src_len, T, eos_id=eos)
            res[mode] = np.array(ids), np.array(lens)
        _ran_as_asked(tr, 2 if mode == "1" and V < 16000 else 0, mode == "1" and give_up)
        tr.close()
        if mode == "any end":
            eos = int(np.array(ids)[0, 2])
    same, near = ((res["0"][0] == res[m][0]).all(axis=1) for m in ("1", "fp32"))
    assert (~near).sum() <= max(1, B // 6)               # (measured: 1 of 3, 1 of 17, 6 of 64, 10 of 100)
    assert (~same).sum() <= (~near).sum()
    np.testing.assert_array_equal(res["0"][1][same], res["1"][1][same])
    assert len(np.unique(res["0"][0])) > 2 and (res["0"][1] < T).any()


@pytest.mark.gpu
@pytest.mark.parametrize("prec,B,S,T,H,E,L", [(0, 20, 9, 6, 64, 24, 2), (1, 33, 12, 7, 128, 64, 3)])
def test_a_captured_step_takes_the_launches(prec, B, S, T, H, E, L, monkeypatch):
    """A step captured into a graph, where no event from outside can be waited for, runs as a launch per layer and position: the same
    kernels as with the loops off, so every replay gives the same bits, whatever ran between them."""
    import torch
    from paper_1802_07170_amd import binding
    cfg = dict(src_vocab=128, tgt_vocab=136, emb=E, hidden=H, layers=L)
    batch = _batch(cfg, B, S, T, seed=B)
    monkeypatch.setenv("CMT_DEC_LOOP", "0")
    _, want, _ = _step(cfg, batch, B, S, T, prec, (0.2, 0.1, 9), loops=False)
    monkeypatch.setenv("CMT_DEC_LOOP", "1")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        tr = binding.Trainer(cfg, B, S, T, precision=prec)
        tr.set_params(I.flatten(I.make_params(cfg, 11, 0.05), cfg))
        tr.set_regularization(0.2, 0.1, 9)
        dev = tr.upload_batch(*batch)
        loss = tr.train_step(dev)
        assert tr.wait_counts() == (2, 0)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            tr.train_step_async(dev)
        for replay in range(4):
            tr.grads.fill_(7.0)
            graph.replay()
            assert abs(tr.fetch_loss() - loss) <= (1e-6 if prec == 0 else 2e-4) * abs(loss)
            np.testing.assert_array_equal(tr.get_grads(), want, err_msg=f"replay {replay}")
            tr.train_step(dev)                            # (eager in between, with its loops)
        assert tr.wait_counts() == (10, 0)
        del graph
        tr.close()
