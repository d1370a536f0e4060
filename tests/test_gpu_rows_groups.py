"""fc_rows_kernel up to 16 images, four lanes to a row: groups of one, two and four blocks (which the test works out) and
what is left of them, rows of no, few and more than sixteen entries side by side, ragged last blocks and block rows."""
import numpy as np
import pytest

import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref

pytestmark = pytest.mark.gpu


def _group(W, bh, bw, workspace):
    """Blocks to a group.  The price of a group falls with every group less and the first of equal ones is taken: four blocks where a
    workgroup has three and more, two where it has two or where 160 KiB of LDS hold the lists and activations (two of each) of no four."""
    M, K = W.shape
    rows, cols = -(-M // bh), -(-K // bw)
    most = max(np.count_nonzero(W[r * bh:(r + 1) * bh, c * bw:(c + 1) * bw]) for r in range(rows) for c in range(cols))
    splits, over = divmod(workspace, rows * 128 * 16 * 4)
    assert over == 0 and 1 <= splits <= cols
    left, tables = -(-cols // splits), 8192
    need = {g: 2 * g * (129 * 16 * 4 + 2 * (-(-(most + 16) // 8) * 8)) for g in (2, 4)}
    assert all(n > 160 * 1024 or n + tables <= 160 * 1024 for n in need.values())        # (whatever the tables take)
    return 4 if left >= 3 and need[4] <= 160 * 1024 else 2 if left >= 2 and need[2] <= 160 * 1024 else 1


@pytest.mark.parametrize("M,K,bh,bw,d,B,group", [(4096, 128 * 17, 128, 128, 0.09, 16, 4), (4096, 128 * 26 - 3, 128, 128, 0.04, 9, 4), (4000, 128 * 41, 128, 128, 0.02, 13, 4),
                                                 (4096, 128 * 33, 128, 128, 0.30, 16, 4), (2050, 96 * 70 + 1, 100, 96, 0.09, 15, 4), (8192, 64 * 40, 64, 64, 0.15, 16, 4),
                                                 (4096, 128 * 9, 128, 128, 0.95, 11, 2), (4096, 128 * 16 - 5, 128, 128, 0.09, 16, 2),
                                                 # one block to a workgroup; LDS for one
                                                 (1000, 121, 128, 128, 0.3, 13, 1), (1000, 128 * 5, 128, 128, None, 16, 1), (700, 128 * 40 - 1, 128, 128, None, 9, 1)])
def test_groups_of_blocks(M, K, bh, bw, d, B, group):
    import torch
    rng = np.random.default_rng(M + K)
    # the density varies from row to row: rows of a step differ in length, some have nothing
    # (None: every weight is there)
    keep = rng.random((M, K)) < (1.0 if d is None else np.minimum(1.0, d * rng.choice([0.0, 0.3, 1.0, 1.7], (M, 1))))
    L = cl.compress_layer((rng.standard_normal((M, K)) * keep).astype(np.float32), 5, 4, bh, bw, upload=True)
    W = cl.decode_layer(L)[3].cpu().numpy()
    assert _group(W, bh, bw, cl.fc_workspace_bytes(L, B, cl.PATH_SPARSE)) == group
    X = np.maximum(rng.standard_normal((B, K)), 0).astype(np.float32)
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda()
    Y = cl.compressed_fc_forward(L, Xd, bd, relu=True, path=cl.PATH_SPARSE)
    assert torch.equal(Y, cl.compressed_fc_forward(L, Xd, bd, relu=True, path=cl.PATH_SPARSE))
    assert_close(Y.cpu().numpy(), fc_ref(W, X, bias), True)
    L.free()
