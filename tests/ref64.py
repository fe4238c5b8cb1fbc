"""The networks in 64 bits, plain torch on the GPU, for tests that need a
reference over many pixels or for values that are not finite."""
from gpu_util import torch_dev


def layers_of(w, shapes):
    """The flat parameters as 64-bit leaves: matrix [out][in], bias, ..."""
    torch = torch_dev()
    v, out, at = torch.from_numpy(w).to("cuda:0").double(), [], 0
    for o, i in shapes:
        out += [v[at:at + o * i].reshape(o, i).clone().requires_grad_(True),
                v[at + o * i:at + o * i + o].clone().requires_grad_(True)]
        at += o * i + o
    return out


def columns(g, L, s):
    """A frame's buffers as [pixels][14], [pixels][k][12], [pixels][16], 64-bit."""
    h, w = g.shape[2:]
    return (g[0].double().reshape(14, -1).t(),
            L[0].double().reshape(L.shape[1], 12, -1).permute(2, 0, 1),
            s.double().expand(h * w, 16))


def glassnet64(flat, G, L, S, relu):
    """[pixels][3], mean pool.  The hidden layer of h is pooled before its affine
    last layer, as the library does (the same in exact arithmetic)."""
    torch = torch_dev()

    def lin(i, x):
        return x @ flat[2 * i].t() + flat[2 * i + 1]

    def mlp(i, x):
        return lin(i + 2, relu(lin(i + 1, relu(lin(i, x)))))
    sigma = mlp(0, torch.cat([G, S], 1))
    act = [(L[:, i, 9:10] > 0).double() for i in range(L.shape[1])]
    Z = sum(a * relu(lin(4, relu(lin(3, torch.cat([L[:, i], sigma], 1))))) for i, a in enumerate(act))
    n = sum(act)
    tau = (Z / n.clamp_min(1.0)) @ flat[10].t() + (n > 0) * flat[11]
    return mlp(9, torch.cat([mlp(6, torch.cat([sigma, tau], 1)), G[:, 11:14]], 1))


def conv64(x, A, b, k):
    """x [h][w][C] -> [h][w][out]: k x k correlation, zero padding; A [out][C k k]."""
    torch = torch_dev()
    h, w, C = x.shape
    A, r = A.reshape(A.shape[0], C, k, k), k // 2
    p = torch.nn.functional.pad(x, (0, 0, r, r, r, r))
    return b + sum(p[i:i + h, j:j + w] @ A[:, :, i, j].t() for i in range(k) for j in range(k))


SR_SHAPES = [(32, 17 * 9), (32, 32 * 9), (3, 32)]
