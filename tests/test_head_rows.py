"""The softmax layer's logits on both of their kernels: a workgroup per four rows with the feature
chunks dealt over its waves (up to 2048 rows), and a wave per two rows walking all chunks.

Bound.  A logit is a sum over D features, each term off by 3 roundings (row scale, product, its
addition within a float4), through at most ceil(D / 256) + 16 further additions (chunks, lanes,
waves, bias); on features that are themselves the layers' fp32 activities, compared through the
layers' own outputs.
"""
import numpy as np
import pytest
import torch

U = 2.0 ** -24


@pytest.mark.gpu
@pytest.mark.parametrize("n,C,d_out", [(1, 10, 256), (3, 2, 260), (4, 2, 2052), (5, 7, 252),
                                       (257, 16, 1284), (2047, 10, 100), (2048, 10, 516),
                                       (2049, 10, 516), (2050, 16, 100)])
def test_logits_rows(n, C, d_out):
    import paper_2404_08573_amd as P
    rng = np.random.default_rng(n + C)
    d_in = 64
    dims = (d_in, 2 * d_out, d_out)  # two feature blocks of different lengths
    layers = [P.Layer(torch.from_numpy(rng.normal(size=(b, a)).astype(np.float32)).cuda(),
                      torch.from_numpy(rng.normal(size=b).astype(np.float32)).cuda())
              for a, b in zip(dims[:-1], dims[1:])]
    D = 3 * d_out
    Wh = rng.normal(size=(C, D)).astype(np.float32)
    bh = rng.normal(size=C).astype(np.float32)
    head = P.Head(torch.from_numpy(Wh).cuda(), torch.from_numpy(bh).cuda())
    x = torch.from_numpy(np.abs(rng.normal(size=(n, d_in))).astype(np.float32)).cuda()
    logits = torch.empty(n, C, device="cuda")
    _, pred = P.ff_head_predict(layers, P.HParams(), head, x, 0, logits=logits)

    h = x.clone()
    h[:, :C] = 0.1
    feats = []
    for L in layers:
        out, g = torch.empty(n, L.W.shape[0], device="cuda"), torch.empty(n, device="cuda")
        P.ff_layer_forward(L, P.HParams(), h, h_out=out, goodness=g)
        torch.cuda.synchronize()
        f = out.cpu().numpy().astype(np.float64)
        feats.append(f / (np.linalg.norm(f, axis=1, keepdims=True) + 1e-8))
        h = out
    A = np.concatenate(feats, axis=1)
    z = A @ Wh.T.astype(np.float64) + bh
    S = A @ np.abs(Wh.T.astype(np.float64)) + np.abs(bh)
    got = logits.cpu().numpy().astype(np.float64)
    # twice the features' own errors: normalised rows by two routes, each within 16 roundings of
    # the same products' sums over at most 2 d_out terms
    k = 3 + -(-D // 256) + 16 + 2 * (16 + 3 * -(-2 * d_out // 16))
    assert (np.abs(got - z) <= k * U * S).all(), (np.abs(got - z) / S).max() / U
    np.testing.assert_array_equal(pred.cpu().numpy(), got.astype(np.float32).argmax(axis=1))
    zs = np.sort(z, axis=1)
    decided = zs[:, -1] - zs[:, -2] > 2 * k * U * S.max(axis=1)
    np.testing.assert_array_equal(pred.cpu().numpy()[decided], z.argmax(axis=1)[decided])
