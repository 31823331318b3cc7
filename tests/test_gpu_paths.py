"""The launches chosen by size (rows per compute unit, parts of a sample, bands of a frame), at the sizes where a rule
turns or a tile ends: against the oracle, or bit for bit against another path that must give the same.  Helpers and
tolerances are those of test_gpu_parity.py.
"""
import numpy as np
import pytest
import torch

from paper_1804_05834_amd import synth
from test_gpu_parity import (CONFIGS, TOL, TOL_BF16, _check_indices, _fill_replay, _replay_step_case, check_argmax, dev, dq, relerr)  # noqa: F401

pytestmark = pytest.mark.gpu


# fp32: parts of 1, 4 and 7 rows per workgroup up to 36, 128 and any number of samples; several samples per workgroup
# above 256.  bf16: one launch for three layers up to 512; fc1 for few rows in 32-row tiles, 64 wide up to 128 rows;
# the head shared by four rows per workgroup from 1024 rows on
@pytest.mark.parametrize("E,K,prec", [(36, 6, 0), (37, 6, 0), (128, 18, 0), (129, 18, 0), (257, 3, 0),
                                      (36, 6, 1), (37, 33, 1), (128, 18, 1), (129, 18, 1), (256, 4, 1), (257, 4, 1),
                                      (512, 18, 1), (513, 18, 1), (1023, 18, 1), (1024, 33, 1), (1027, 1, 1)])
def test_act_where_the_launches_change(dq, orc, E, K, prec):
    print("case act", E, K, prec, flush=True)
    tol = TOL_BF16 if prec else TOL
    m = dq.Dqn(dq.make_config(num_actions=K, dueling=1, max_act_batch=E, precision=prec))
    p = synth.he_uniform_params(3 + K, K, 1, bias_scale=0.05)
    m.set_params(0, torch.from_numpy(p))
    obs = synth.states(31, E)
    a, q = m.act(dev(obs), 0.0, 99, want_q=True)
    q, ref = q.cpu().numpy(), orc.forward(p, K, 1, obs.numpy(), quant=prec)
    # row by row, so that none hides behind the largest; with one action a row has a single value, which may lie
    # near zero while the sums behind it do not: the scale of such a row is that of all values (their rms)
    scale = np.maximum(np.abs(ref).max(axis=1), np.sqrt(np.mean(ref ** 2)))
    assert np.all(np.abs(q - ref).max(axis=1) <= tol * scale)
    check_argmax(a.cpu().numpy(), ref, tol)
    m.close()


# up to two observations fc1 and the head are one launch, with the counter of its workgroups cleared by the conv launch:
# several calls in a row, the counts of observations mixed, Q and actions of each
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("K,dueling", [(1, 0), (18, 1), (31, 1), (64, 1)])
def test_act_on_few_observations(dq, orc, K, dueling, prec):
    print("case act on few", K, dueling, prec, flush=True)
    tol = TOL_BF16 if prec else TOL
    m = dq.Dqn(dq.make_config(num_actions=K, dueling=dueling, max_act_batch=3, precision=prec))
    p = synth.he_uniform_params(3 + K, K, dueling, bias_scale=0.05)
    m.set_params(0, torch.from_numpy(p))
    obs = synth.states(31, 3)
    ref = orc.forward(p, K, dueling, obs.numpy(), quant=prec)
    on = dev(obs)
    got = [(E, m.act(on[3 - E:], 0.0, 99, want_q=True)) for E in (1, 2, 1, 3, 2, 1)]
    for E, (a, q) in got:
        r = ref[3 - E:]
        scale = np.maximum(np.abs(r).max(axis=1), np.sqrt(np.mean(ref ** 2)))
        assert np.all(np.abs(q.cpu().numpy() - r).max(axis=1) <= tol * scale), E
        check_argmax(a.cpu().numpy(), r, tol)
    m.close()

# up to 18 observations (7 parts each, two workgroups per part on 256 compute units) conv3's channels are split over two
# workgroups in fp32; 19 and 36 are one workgroup per part.  The sums are the same, so the bits are
@pytest.mark.parametrize("prec", [0, 1])
def test_act_same_bits_however_many(dq, prec):
    m = dq.Dqn(dq.make_config(num_actions=6, dueling=1, max_act_batch=36, precision=prec))
    m.set_params(0, torch.from_numpy(synth.he_uniform_params(8, 6, 1, bias_scale=0.05)))
    on = dev(synth.states(33, 36))
    a36, q36 = (t.clone() for t in m.act(on, 0.0, 99, want_q=True))
    for E in (1, 2, 3, 17, 18, 19):
        print("case act same bits", prec, E, flush=True)
        a, q = m.act(on[36 - E:], 0.0, 99, want_q=True)
        assert torch.equal(q, q36[36 - E:]) and torch.equal(a, a36[36 - E:]), E
    m.close()


# bf16: up to an observation per compute unit the conv layers are units of one workgroup each, above it the pipeline of waves;
# fc1's tiles are the same up to 511 rows
def test_act_same_bits_where_the_conv_launch_changes(dq):
    m = dq.Dqn(dq.make_config(num_actions=6, dueling=1, max_act_batch=511, precision=1))
    m.set_params(0, torch.from_numpy(synth.he_uniform_params(8, 6, 1, bias_scale=0.05)))
    on = synth.frames(3, torch.arange(4 * 511, device="cuda"), device="cuda").view(511, 4, 84, 84)
    a511, q511 = (t.clone() for t in m.act(on, 0.0, 99, want_q=True))
    for E in (37, 128, 255, 256, 257, 510):
        print("case act same bits, conv launches", E, flush=True)
        a, q = m.act(on[511 - E:], 0.0, 99, want_q=True)
        assert torch.equal(q, q511[511 - E:]) and torch.equal(a, a511[511 - E:]), E
    m.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("K,dueling,small", [(18, 1, 0), (4, 0, 0), (64, 1, 0), (18, 1, 1)])
def test_an_observation_has_the_same_bits_alone_and_among_others(dq, K, dueling, small, prec):
    """One and two observations take launches of their own behind the conv layers; every sum is that of the launches for
    more: up to 36 in fp32 (the conv layers of more are summed in other parts) and 511 in bf16.  small: fc1's weights are subnormal, the head's bring its sums back."""
    print("case bits of few", K, dueling, small, prec, flush=True)
    T = {name: synth.u24(70 + i, torch.arange(int(np.prod(shape)))).numpy().reshape(shape) - 0.5 if name.endswith(".W") else
         np.zeros(shape) for i, (name, shape, _) in enumerate(synth.param_spec(K, dueling))}
    if small:
        T["fc1.W"] *= 1e-39
        T["A.W"] *= 1e30
        T["V.W"] *= 1e30
    else:
        T["fc1.b"] += 0.01
    blob = np.concatenate([T[n].astype(np.float32).ravel() for n, _, _ in synth.param_spec(K, dueling)])
    n = 511 if prec else 36
    m = dq.Dqn(dq.make_config(num_actions=K, dueling=dueling, max_act_batch=n, precision=prec))
    m.set_params(0, torch.from_numpy(blob))
    obs = dev(synth.states(31, n))
    a, q = m.act(obs, 0.0, 99, want_q=True)
    assert torch.isfinite(q).all() and q.unique().numel() > n
    for E in (1, 2, 3):
        for i in range(0, n - E + 1, 5):
            for static in (False, True):
                x, y = m.act(obs[i:i + E].contiguous(), 0.0, 99, want_q=True, static=static)
                assert torch.equal(y, q[i:i + E]) and torch.equal(x, a[i:i + E]), (E, i, static)
    m.close()


# fp32 steps: parts of the samples of s' are 1 row up to 14, 4 rows above; those of s are 2 rows up to 32, 4 rows above;
# conv1 sums its frames in two halves up to 34; one launch for the conv layers up to 42; from 60 up to 128 one for s' and
# layers for s
@pytest.mark.parametrize("B", [14, 15, 34, 35, 42, 43, 59, 60, 128, 129])
def test_fp32_step_where_the_launches_change(dq, orc, B):
    print("case fp32 step", B, flush=True)
    _replay_step_case(dq, orc, cap=30000, B=B, draw_seed=41)


@pytest.mark.parametrize("prec,B", [(1, 31), (1, 85), (1, 86), (1, 170), (1, 171)])
def test_bf16_step_where_the_launches_change(dq, orc, prec, B):
    """bf16: one launch for the conv layers up to 85 (256 samples of three passes), the large fc1 tiles from 512 rows on."""
    print("case bf16 step", B, flush=True)
    _replay_step_case(dq, orc, cap=30000, B=B, draw_seed=41, tol=TOL_BF16, prec=1)


@pytest.mark.parametrize("B,cus", [(1, 2), (2, 9), (4, 7), (5, 7), (75, 9), (100, 65), (110, 65), (127, 40), (129, 100)])
def test_conv_backward_over_ranges_of_samples(dq, monkeypatch, B, cus):
    """bf16: the conv layers' gradients with one to 37 samples in a workgroup (pairs of samples and single ones in conv3's input
    gradient) against few: the same activations, and sums of the same products split another way, to the fp32 path's tolerance."""
    print("case conv backward", B, cus, flush=True)
    batch = tuple(dev(t) for t in synth.batch(29, B, 18))
    got = []
    for n in (None, cus):
        if n:
            monkeypatch.setenv("DQN_COMPUTE_UNITS", str(n))
        m = dq.Dqn(dq.make_config(max_batch=B, precision=1, seed=7, **CONFIGS["dueling_ddqn"]))
        m.train_step(B, batch)
        got.append((m.get_activations(3, B), m.get_params(2).cpu().numpy()))
        m.close()
    assert torch.equal(got[0][0], got[1][0])
    lo = 0
    for name, n in (("conv1", 8224), ("conv2", 32832), ("conv3", 36928)):
        assert relerr(got[1][1][lo:lo + n], got[0][1][lo:lo + n]) <= TOL, name
        lo += n


@pytest.mark.parametrize("n", [35, 42])
def test_fp32_step_activations_are_those_of_the_separate_launches(dq, n):
    """A batch of 43 runs the layers of s as launches of their own, its first n rows alone as units of one launch: the
    stored activations, which the ReLU decisions are taken on, must have the same bits."""
    print("case activations", n, flush=True)
    K = 18
    batch = tuple(dev(t) for t in synth.batch(11, 43, K))
    acts = []
    for B in (43, n):
        m = dq.Dqn(dq.make_config(max_batch=B, seed=7, **CONFIGS["dueling_ddqn"]))
        m.train_step(B, tuple(t[:B].contiguous() for t in batch))
        acts.append([m.get_activations(layer, n) for layer in (1, 2, 3)])
        m.close()
    for layer, (x, y) in enumerate(zip(*acts)):
        assert torch.equal(x, y), layer + 1


@pytest.mark.parametrize("n", [4095, 4096, 4097, 8193])
def test_tree_build_at_block_edges(dq, orc, n):
    print("case tree build", n, flush=True)
    m = dq.Dqn(dq.make_config(replay_capacity=9000))
    p = synth.exp_priorities(9, n)
    for _ in range(2):   # the second build finds the arrival counter as the first left it
        m.per_fill(dev(p))
        ref = orc.tree_build(p.numpy(), m.L, float(np.float32(0.6)))
        assert np.array_equal(m.tree.cpu().numpy()[1:], ref[1:])
    for B in (1, 5, 1023):
        idx, w = m.per_sample(B, 0.4, 4242)
        idx_ref, w_ref = _check_indices(orc, idx.cpu().numpy(), ref, n, B, 0.4, 4242)
        same = idx.cpu().numpy() == idx_ref
        assert same.mean() > 0.99 and relerr(w.cpu().numpy()[same], w_ref[same]) <= TOL
    m.close()


@pytest.mark.parametrize("cap", [16, 31, 1028])
def test_store_at_the_edges_of_the_ring(dq, orc, cap):
    """Rings that a call nearly fills, and runs that end, begin and wrap at the ring's last slot."""
    print("case store", cap, flush=True)
    m = dq.Dqn(dq.make_config(replay_capacity=cap))
    ref = orc.ReplayState(cap, float(np.float32(0.6)))
    pos, most = 0, min(1020, cap - 8)
    for n in (1, most, 1, 7, most, most, 2, cap % 7 + 1, most):
        fr = synth.frames(21, torch.arange(pos, pos + n, device="cuda"), device="cuda")
        d = synth.dones(42, n, 0.05, "cuda", first=pos)
        m.replay_store(fr, synth.actions(40, n, 18, "cuda", first=pos), synth.rewards(41, n, "cuda", first=pos), d)
        ref.store(d.cpu().numpy())
        pos += n
        assert np.array_equal(m.tree.cpu().numpy()[1:], ref.tree[1:]), pos
        assert m.replay_state() == (pos % cap, min(pos, cap), pos)
    m.close()


# bands of a frame; widths that leave every row at another alignment; a frame too tall for LDS; the smallest
@pytest.mark.parametrize("n,H,W", [(1, 210, 160), (3, 210, 161), (300, 97, 37), (2, 336, 640), (2, 337, 100), (5, 1, 1), (2, 83, 1)])
def test_preprocess_shapes(dq, orc, n, H, W):
    print("case preprocess", n, H, W, flush=True)
    raw = (synth.u24(61, torch.arange(n * H * W)) * 256).floor().clamp(max=255).to(torch.uint8).reshape(n, H, W)
    lut = (255.0 * synth.u24(62, torch.arange(256))).float()
    for table in (lut, None):
        out = dq.preprocess(raw.cuda(), None if table is None else table.cuda()).cpu().numpy()
        ref, val = orc.preprocess(raw.numpy(), None if table is None else table.numpy())
        diff = out.astype(np.int32) - ref.astype(np.int32)
        near = np.abs(val - np.floor(val) - 0.5) <= 1e-3   # (as in test_preprocess_parity)
        assert np.all(diff[~near] == 0) and np.all(np.abs(diff) <= 1)


@pytest.mark.parametrize("replay,units", [(False, 64), (True, 64), (False, 199), (True, 37)])
def test_fp32_workgroups_that_take_samples_of_both_networks(dq, monkeypatch, replay, units):
    """The passes over s' of a batch of 100 are 200 whole samples, the first half through the online network, the second
    through the target network.  Planned for fewer compute units than that, a workgroup takes several and passes from one
    network to the other (with biases of its own): the same sums in the same order as with a workgroup per sample."""
    print("case both networks in a workgroup", replay, units, flush=True)
    B, K, cap = 100, 18, 5000
    got = []
    for limit in (None, units):
        monkeypatch.delenv("DQN_COMPUTE_UNITS", raising=False)
        if limit:
            monkeypatch.setenv("DQN_COMPUTE_UNITS", str(limit))
        m = dq.Dqn(dq.make_config(max_batch=B, replay_capacity=cap if replay else 0, seed=7, **CONFIGS["dueling_ddqn"]))
        for net in (0, 1):
            m.set_params(net, torch.from_numpy(synth.he_uniform_params(5 + net, K, 1, bias_scale=0.5)))
        if replay:
            _fill_replay(m, cap, K=K)
            m.per_fill(synth.exp_priorities(9, cap, "cuda"))
            outs = [m.train_step(B, None, draw_seed=3)]
        else:
            batch = tuple(dev(t) for t in synth.batch(11, B, K))
            outs = [m.train_step(B, batch)]
        got.append(outs)
        m.close()
    for x, y in zip(*got):
        for name in ("q_next_online", "q_next_target", "a_star", "y") + (("idx", "is_w") if replay else ()):
            assert torch.equal(x[name], y[name]), name


@pytest.mark.parametrize("E,B", [(3, 8), (60, 32), (300, 64), (1, 160)])
def test_fp32_parameters_written_in_place(dq, E, B):
    """fp32 has no copies of the weights: what a caller writes into its own parameter buffers (another context's contents, a
    target moved towards the online network) is what the next call uses, in every launch, and nothing in the workspace has
    to survive from one call to the next."""
    print("case parameters in place", E, B, flush=True)
    K = 18
    cfg = dict(max_batch=B, max_act_batch=E, **CONFIGS["dueling_ddqn"])
    obs, batch = dev(synth.states(31, E)), tuple(dev(t) for t in synth.batch(11, B, K))
    m, n = dq.Dqn(dq.make_config(seed=7, **cfg)), dq.Dqn(dq.make_config(seed=8, target_seed=9, **cfg))
    for name in ("online", "target", "opt_state"):
        n._bufs[name].copy_(m._bufs[name])
    on, tg = m.get_params(0), m.get_params(1)
    m.set_params(1, 0.5 * on + 0.5 * tg)   # the same in the canonical order
    for buf in (n._bufs["target"].view(torch.float32),):
        buf.copy_(0.5 * n._bufs["online"].view(torch.float32) + 0.5 * buf)
    for step in range(2):
        n._bufs["workspace"].fill_(255)
        a, q = m.act(obs, 0.0, 5, want_q=True)
        b, p = n.act(obs, 0.0, 5, want_q=True)
        assert torch.equal(q, p) and torch.equal(a, b), step
        n._bufs["workspace"].fill_(255)
        x, y = m.train_step(B, batch), n.train_step(B, batch)
        for name in x:
            assert torch.equal(x[name], y[name]), (step, name)
        for which in (0, 1, 2, 3):
            assert torch.equal(m.get_params(which), n.get_params(which)), (step, which)
    m.close()
    n.close()


@pytest.mark.parametrize("B", [14, 30, 64, 100])
@pytest.mark.parametrize("layer", [2, 3])
def test_fp32_split_products_are_no_less_exact_than_the_fp32_chain(dq, layer, B):
    """conv2 and conv3 in the split form (the passes over s') against the plain fp32 chain (the pass on s) on the same states:
    the error against fp64, rms over the outputs.  Inputs and outputs of the layer are read off exactly: conv1 is one
    pixel times a 16-bit weight per channel, the other conv layer and the head pass single values on."""
    print("case split exactness", layer, B, flush=True)
    K = 64
    rng = np.random.default_rng(100 * layer + B)
    T = {name: np.zeros(shape) for name, shape, _ in synth.param_spec(K, 0)}
    taps = [(rng.integers(4), rng.integers(8), rng.integers(8)) for _ in range(32)]
    w1 = rng.integers(32768, 65536, 32) / 65536.0 * np.where(rng.random(32) < 0.3, -1, 1)   # a third: nothing after the ReLU
    for o in range(32):
        T["conv1.W"][(o,) + taps[o]] = w1[o]
    for o in range(64):
        T["conv2.W"][o, o % 32, 1 + o // 32, 2] = 1.0
        T["conv3.W"][o, o, 1, 1] = 1.0
    name, fan = ("conv2.W", 512) if layer == 2 else ("conv3.W", 576)
    T[name] = np.where(rng.random(T[name].shape) < 0.2, rng.normal(0, (6.0 / fan) ** 0.5, T[name].shape), 0)
    pick = rng.permutation(3136)[:K]
    T["fc1.W"][np.arange(K), pick] = T["A.W"][np.arange(K), np.arange(K)] = 1.0
    blob = torch.from_numpy(np.concatenate([T[n].astype(np.float32).ravel() for n, _, _ in synth.param_spec(K, 0)]))
    s, _, a, r, d = synth.batch(11, B, K)
    m = dq.Dqn(dq.make_config(num_actions=K, dueling=0, max_batch=B))
    m.set_params(0, blob)
    m.set_params(1, blob)
    out = m.train_step(B, tuple(dev(t) for t in (s, s, a, r, d)))
    # the layer's inputs in fp32: integer sums, exact, times fp32(1 / 255)
    h = np.zeros((B, 32, 20, 20), np.float32)
    for o, (c, y, x) in enumerate(taps):
        v = (s[:, c, y:y + 77:4, x:x + 77:4].numpy().astype(np.float64) * w1[o]).astype(np.float32)
        h[:, o] = np.maximum(v * np.float32(1.0 / 255.0), 0)

    def conv(v, name, stride):
        W = torch.from_numpy(T[name].astype(np.float32)).double()
        n = (v.shape[2] - W.shape[-1]) // stride + 1
        u, W = torch.nn.functional.unfold(v, W.shape[-1], stride=stride), W.reshape(64, -1)
        return torch.matmul(W, u).reshape(B, 64, n, n), torch.matmul(W.abs(), u.abs()).reshape(B, 64, n, n)

    y, mag = conv(torch.from_numpy(h).double(), "conv2.W", 2)
    if layer == 3:
        y, mag = conv(y, "conv3.W", 1)
    else:
        y, mag = y[:, :, 1:8, 1:8], mag[:, :, 1:8, 1:8]
    y, mag = y.flatten(1)[:, pick], mag.flatten(1)[:, pick]
    on = y > 0
    rms = {k: float((((out[k].cpu().double() - y) / mag)[on] ** 2).mean().sqrt()) for k in ("q_s", "q_next_online", "q_next_target")}
    assert rms["q_s"] < 1e-7   # what was read off is the layer
    assert max(rms["q_next_online"], rms["q_next_target"]) <= rms["q_s"], rms
    m.close()


def _positive_network(K):
    """All weights and biases positive: an infinity anywhere reaches the Q-values as one."""
    T = {name: np.abs(synth.u24(50 + i, torch.arange(int(np.prod(shape)))).numpy() - 0.5).reshape(shape) + 0.01
         for i, (name, shape, _) in enumerate(synth.param_spec(K, 0))}
    return T, lambda: torch.from_numpy(np.concatenate([T[n].astype(np.float32).ravel() for n, _, _ in synth.param_spec(K, 0)]))


@pytest.mark.parametrize("where,value", [("conv1.b", np.inf), ("conv1.W", np.inf), ("conv2.W", np.inf), ("conv2.b", np.inf), ("conv3.W", np.inf),
                                         ("conv2.W", -np.inf), ("conv3.b", np.nan), ("conv1.W", 1e36), (None, 0)])
def test_infinities_pass_through_the_fp32_conv_layers(dq, where, value):
    """An infinite weight or activation, or a sum that overflows, is in the split form (acting, the passes over s') what it is
    in the plain fp32 chain (the pass on s)."""
    print("case infinities", where, value, flush=True)
    K = 5
    T, blob = _positive_network(K)
    if where:
        T[where].reshape(-1)[T[where].size // 2 + 3] = value
    for B in (14, 30, 64):
        s, _, a, r, d = synth.batch(11, B, K)
        s = s.clamp(min=1)   # no zero for an infinite weight to meet
        m = dq.Dqn(dq.make_config(num_actions=K, dueling=0, max_batch=B, max_act_batch=300))
        for net in (0, 1):
            m.set_params(net, blob())
        acted = [m.act(dev(s)[:E].contiguous(), 0.0, 1, want_q=True)[1] for E in (3, B)]
        acted.append(m.act(dev(s).repeat(300 // B + 1, 1, 1, 1)[:300].contiguous(), 0.0, 1, want_q=True)[1][:B])
        out = m.train_step(B, tuple(dev(t) for t in (s, s, a, r, d)))
        ref = out["q_s"]
        assert bool(torch.isfinite(ref).all()) == (where is None or value < 0 or np.isnan(value))
        for q in (out["q_next_online"], out["q_next_target"], acted[0], acted[1], acted[2]):
            x = ref[:q.shape[0]]
            assert torch.equal(torch.isinf(q), torch.isinf(x)) and torch.equal(torch.isnan(q), torch.isnan(x))
            fin = torch.isfinite(x)
            assert bool(((q - x).abs()[fin] <= TOL * x.abs()[fin]).all())
        m.close()


def test_infinite_gradients_of_small_fp32_steps(dq, monkeypatch):
    """An infinite TD error: the gradients of conv2 and conv1 in the one-launch split form (a batch of 32) and by the layers'
    own launches (the same planned for fewer compute units) are infinite, and NaN, in the same places."""
    print("case infinite gradients", flush=True)
    B, K = 32, 5
    _, blob = _positive_network(K)
    s, sn, a, r, d = synth.batch(11, B, K)
    s = s.clamp(min=1)
    r[3] = float("inf")
    got = []
    for limit in (None, 100):
        if limit:
            monkeypatch.setenv("DQN_COMPUTE_UNITS", str(limit))
        m = dq.Dqn(dq.make_config(num_actions=K, dueling=0, double_q=0, loss_kind=0, max_batch=B))
        for net in (0, 1):
            m.set_params(net, blob())
        m.train_step(B, tuple(dev(t) for t in (s, sn, a, r, d)))
        got.append(m.get_params(2))
        m.close()
    x, y = got
    assert torch.isinf(y).any()
    n = 77984   # conv1 to conv3
    for k, f in (("inf", torch.isinf), ("nan", torch.isnan)):
        assert torch.equal(f(x[:n]), f(y[:n])), (k, int(f(x[:n]).sum()), int(f(y[:n]).sum()))


@pytest.mark.parametrize("E,B", [(3, 8), (300, 77), (600, 200)])
def test_bf16_context_from_copied_buffers(dq, E, B):
    """bf16: the parameter, optimizer and shadow buffers of one context, copied into another's, make it the same network in
    every launch; nothing in the workspace has to survive from one call to the next."""
    print("case copied buffers", E, B, flush=True)
    K = 18
    cfg = dict(max_batch=B, max_act_batch=E, precision=1, **CONFIGS["dueling_ddqn"])
    obs, batch = dev(synth.states(31, E)), tuple(dev(t) for t in synth.batch(11, B, K))
    m, n = dq.Dqn(dq.make_config(seed=7, **cfg)), dq.Dqn(dq.make_config(seed=8, target_seed=9, **cfg))
    m.train_step(B, batch)
    for name in ("online", "target", "opt_state", "shadow_bf16"):
        n._bufs[name].copy_(m._bufs[name])
    for step in range(3):
        if step == 2:
            m.sync_target()
            n.sync_target()
        n._bufs["workspace"].fill_(255)
        a, q = m.act(obs, 0.0, 5, want_q=True)
        b, p = n.act(obs, 0.0, 5, want_q=True)
        assert torch.equal(q, p) and torch.equal(a, b), step
        n._bufs["workspace"].fill_(255)
        x, y = m.train_step(B, batch), n.train_step(B, batch)
        for name in x:
            assert torch.equal(x[name], y[name]), (step, name)
        for which in (0, 1, 2, 3):
            assert torch.equal(m.get_params(which), n.get_params(which)), (step, which)
    m.close()
    n.close()


@pytest.mark.parametrize("prec,E,B", [(0, 1, 5), (0, 130, 32), (0, 40, 100), (1, 3, 33), (1, 2100, 77)])
def test_launches_with_no_more_lds_than_every_workgroup_gets(dq, orc, monkeypatch, prec, E, B):
    print("case small lds", prec, E, B, flush=True)
    monkeypatch.setenv("DQN_SMALL_LDS", "1")
    K, tol = 18, TOL_BF16 if prec else TOL
    m = dq.Dqn(dq.make_config(num_actions=K, dueling=1, max_act_batch=E, precision=prec))
    p = synth.he_uniform_params(3 + K, K, 1, bias_scale=0.05)
    m.set_params(0, torch.from_numpy(p))
    obs = synth.states(31, E)
    q = m.act(dev(obs), 0.0, 99, want_q=True)[1].cpu().numpy()
    rows = np.unique(np.linspace(0, E - 1, 200).astype(int))
    ref = orc.forward(p, K, 1, obs.numpy()[rows], quant=prec)
    assert relerr(q[rows], ref) <= tol
    if E <= 32:
        assert np.array_equal(m.act(dev(obs), 0.0, 99, want_q=True, static=True)[1].cpu().numpy(), q)
    m.close()
    _replay_step_case(dq, orc, cap=30000, B=B, draw_seed=41, tol=tol, prec=prec)


@pytest.mark.parametrize("B,cus", [(135, None), (136, 7), (211, 3), (449, None), (600, 31)])
def test_conv_layers_of_many_rows_with_weights_in_lds(dq, monkeypatch, B, cus):
    """fp32: the same bits as the tiled launches, which run where a workgroup gets no more LDS than every one does."""
    print("case rows", B, cus, flush=True)
    got = []
    batch = tuple(dev(t) for t in synth.batch(17, B, 18))
    if cus:
        monkeypatch.setenv("DQN_COMPUTE_UNITS", str(cus))
    for small in ("0", "1"):
        monkeypatch.setenv("DQN_SMALL_LDS", small)
        m = dq.Dqn(dq.make_config(max_batch=B, seed=7, **CONFIGS["dueling_ddqn"]))
        out = m.train_step(B, batch)
        got.append([out[k] for k in ("q_s", "q_next_online", "q_next_target", "td")] + [m.get_params(2)])
        m.close()
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.parametrize("B", [131, 170, 171, 347, 513, 700])
def test_fc1_in_tiles_of_any_height(dq, monkeypatch, B):
    """fp32, 7, 2 and 1 splits: the number of compute units moves the tiles' height (48 to 128 rows), never a bit; and the
    hidden layer lies within the error of a sum of 3136 products, K 2^-24 sum |x w|, of float64."""
    print("case fc1 tiles", B, flush=True)
    batch = tuple(dev(t) for t in synth.batch(23, B, 18))
    first = None
    for cus in (256, 230, 200, 160, 130, 100, 80, 60):
        monkeypatch.setenv("DQN_COMPUTE_UNITS", str(cus))
        m = dq.Dqn(dq.make_config(max_batch=B, seed=7, **CONFIGS["dueling_ddqn"]))
        p = m.get_params(0).cpu().double()
        out = m.train_step(B, batch)
        got = [m.get_activations(4, B)] + [out[k] for k in ("q_s", "q_next_online", "q_next_target")]
        x = m.get_activations(3, B)
        m.close()
        if first is None:
            first = got
            o = 32 * 256 + 32 + 64 * 512 + 64 + 64 * 576 + 64
            w, b = p[o:o + 512 * 3136].view(512, 3136), p[o + 512 * 3136:o + 512 * 3136 + 512]
            x = x.cpu().double().view(B, 3136)
            err = (got[0].cpu().double() - (x @ w.T + b).clamp(min=0)).abs()
            assert (err <= 3136 * 2.0 ** -24 * (x.abs() @ w.abs().T + b.abs())).all()
        for a, c in zip(first, got):
            assert torch.equal(a, c)


@pytest.mark.parametrize("B", [420, 463, 492, 607, 778, 1000])
def test_backward_on_one_stream_and_on_three(dq, monkeypatch, B):
    """fp32: the layers' own backward launches of the largest batches and the launches with both gradients of a layer, which one
    stream takes at every batch, add in the same order: the same bits (the head's weight gradient is split another way)."""
    print("case streams", B, flush=True)
    batch = tuple(dev(t) for t in synth.batch(29, B, 18))
    got = []
    for single in ("0", "1"):
        monkeypatch.setenv("DQN_SINGLE_STREAM", single)
        m = dq.Dqn(dq.make_config(max_batch=B, seed=7, **CONFIGS["dueling_ddqn"]))
        m.train_step(B, batch)
        got.append([m.get_params(k)[:1684128] for k in (0, 2)])
        m.close()
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.parametrize("B", [129, 191, 193, 419, 421])
def test_input_gradient_tiles_at_their_edges(dq, orc, B):
    """fp32: tiles of 64 rows of fc1's, conv3's and conv2's input gradients, in both schedules, against the oracle."""
    print("case input gradient tiles", B, flush=True)
    _replay_step_case(dq, orc, cap=30000, B=B, draw_seed=41)


def test_fc1_with_two_and_four_stages_in_lds(dq, monkeypatch):
    """bf16, 750 samples in each of three passes: the same sums whatever the number of stages, behind the same conv launches."""
    print("case fc1 stages", flush=True)
    B, K, got = 750, 18, []
    batch = tuple(dev(t) for t in synth.batch(11, B, K))
    monkeypatch.setenv("DQN_CONV12_MIN_SAMPLES", "1000000")
    monkeypatch.setenv("DQN_FUSED_BWD", "0")
    for small in ("0", "1"):
        monkeypatch.setenv("DQN_SMALL_LDS", small)
        m = dq.Dqn(dq.make_config(max_batch=B, precision=1, seed=7, **CONFIGS["dueling_ddqn"]))
        out = m.train_step(B, batch)
        got.append([out[k] for k in ("q_s", "q_next_online", "q_next_target", "td")] + [m.get_params(2)])
        m.close()
    for x, y in zip(*got):
        assert torch.equal(x, y)
