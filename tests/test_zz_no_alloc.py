"""cmt_eval_loss_static (the entry point that allocates nothing: every intermediate lives in a static
device array of the library) against cmt_eval_loss (intermediates in the caller's workspace): same
kernels in the same order, so the loss must be bit-identical and the token count equal — on two
calls in a row, the second with a smaller input, in both precisions; a shape whose intermediates do
not fit the array is refused with a clear message and leaves the handle usable."""
import numpy as np
import pytest

from paper_1802_07170_amd import inputs as I

pytestmark = pytest.mark.gpu


def _case(prec):
    from paper_1802_07170_amd import binding
    c = I.CONFIGS["tiny"]
    cfg = I.model_cfg(c)
    params = I.make_params(cfg, c["seed"])
    big = I.make_batch(c)                                        # 8 sentences x 10 tokens
    small = I.make_batch(c, batch=5, len_range=(3, 7), seed=11)  # ragged, fewer and shorter sentences
    tr = binding.Trainer(cfg, 8, 10, 10, precision=prec)
    try:
        tr.set_params(I.flatten(params, cfg))
        dev_big, dev_small = tr.upload_batch(*big), tr.upload_batch(*small)
        want_big, want_small = tr.eval_loss(dev_big), tr.eval_loss(dev_small)
        # a training step in between: its gradients and intermediates must survive the static calls
        loss_train = tr.train_step(dev_big)
        grads = tr.get_grads()
        h_o = tr.debug_fetch("h_o", (10, tr.padded_batch(), cfg["hidden"]))
        got_big = tr.eval_loss_static(dev_big)
        got_small = tr.eval_loss_static(dev_small)
        assert got_big == want_big, (got_big, want_big)
        assert got_small == want_small, (got_small, want_small)
        assert got_big[1] == float(big[3].sum()) and got_small[1] == float(small[3].sum())
        assert np.isfinite(got_big[0]) and abs(got_big[0] - np.log(1000.0)) < 0.1
        # the handle's own state is untouched
        assert np.array_equal(tr.get_grads(), grads)
        assert np.array_equal(tr.debug_fetch("h_o", h_o.shape), h_o)
        assert tr.train_step(dev_big) == loss_train
        # and once more after the step, larger input after the smaller one
        assert tr.eval_loss_static(dev_big) == want_big
    finally:
        tr.close()


def test_static_eval_matches_workspace_eval_fp32():
    _case(0)


def test_static_eval_matches_workspace_eval_bf16():
    _case(1)


@pytest.mark.parametrize("H,E,L,length,prec", [(64, 64, 2, 45, 0), (80, 64, 4, 36, 1)])
def test_static_eval_takes_shapes_that_just_fit(H, E, L, length, prec):
    from paper_1802_07170_amd import binding
    cfg = dict(src_vocab=1000, tgt_vocab=1000, emb=E, hidden=H, layers=L)
    batch = I.make_batch(dict(cfg, ids="zipf", batch=16, len_range=(length, length), seed=4))
    tr = binding.Trainer(cfg, 16, length, length, precision=prec)
    try:
        tr.init_params(1, 0.1)
        dev = tr.upload_batch(*batch)
        assert tr.eval_loss_static(dev) == tr.eval_loss(dev)
    finally:
        tr.close()


@pytest.mark.parametrize("H,E,L,B,S,T", [(128, 64, 2, 20, 12, 9), (80, 64, 3, 40, 9, 6), (48, 24, 4, 17, 20, 5), (256, 64, 1, 16, 6, 3),
                                         (16, 8, 2, 33, 7, 7), (64, 32, 2, 70, 5, 1)])
@pytest.mark.parametrize("prec", [0, 1])
def test_static_eval_is_the_workspace_eval_bit_by_bit(H, E, L, B, S, T, prec):
    """Several networks per shape, at weights of a scale where another order of the sums shows in the loss."""
    from paper_1802_07170_amd import binding
    cfg = dict(src_vocab=504, tgt_vocab=504, emb=E, hidden=H, layers=L)
    recipe = dict(cfg, ids="zipf", batch=B, seed=H)
    batch = I.make_batch(recipe, len_range=(max(1, S // 2), S))[:2] + I.make_batch(recipe, len_range=(max(1, T // 2), T))[2:]
    tr = binding.Trainer(cfg, B, S, T, precision=prec)
    try:
        dev = tr.upload_batch(*batch)
        for seed in range(6):
            tr.init_params(seed, 4.0 / H ** 0.5)
            assert tr.eval_loss_static(dev) == tr.eval_loss(dev), seed
    finally:
        tr.close()


def test_static_eval_refuses_a_shape_beyond_the_array():
    from paper_1802_07170_amd import binding
    c = I.CONFIGS["small"]                                       # vocabulary 32000: the slab buffers alone exceed the array
    cfg = I.model_cfg(c)
    batch = I.make_batch(c, batch=4, len_range=(5, 8), seed=3)
    tr = binding.Trainer(cfg, 4, 8, 8, precision=1)
    try:
        tr.init_params(1, 0.1)
        dev = tr.upload_batch(*batch)
        want = tr.eval_loss(dev)
        with pytest.raises(binding.CmtError) as e:
            tr.eval_loss_static(dev)
        assert e.value.code == binding.CMT_EINVAL and "static buffer holds" in str(e.value)
        assert tr.eval_loss(dev) == want                         # still usable
    finally:
        tr.close()
