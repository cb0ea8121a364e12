"""Kernels at the sizes where their tiles, parts and dispatch rules change,
against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import field as ofield
from parity import check_mag

pytestmark = pytest.mark.gpu


def _t(torch, dev, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


# sixteen levels that each fit one bin of 8192 entries (the largest a level may have)
SMALL_TABLES = dataclasses.replace(W.C2_FIELD, log2_table=13, max_res=256)


@pytest.mark.parametrize("spec,S", [(W.C1_FIELD, 64), (W.C1_FIELD, 226), (W.C1_FIELD, 1023), (W.C1_FIELD, 1025),
                                    (W.C1_FIELD, 131073), (SMALL_TABLES, 16), (SMALL_TABLES, 3001)],
                         ids=["sorted", "one-part", "one-used", "two-used", "all-parts", "16-sorted", "16-levels"])
def test_scatter_of_single_bin_levels(nsl, gpu, spec, S):
    """nsl_encode_bwd where every level fits one bin: too few samples for a
    part (the counting sort), one part, parts of unequal size, every part;
    overwriting and accumulating, at 1e-5 (FP32 values) and 2e-2 (BF16)."""
    import torch
    f = nsl.Field(spec)
    nt = f.layout["table_floats"]
    rng = np.random.default_rng(S)
    xn = rng.uniform(size=(S, 3)).astype(np.float32)
    xn[: S // 2] = np.clip(0.4 + 1e-3 * np.arange(S // 2)[:, None] / max(1, S // 2), 0, 1)    # runs in shared cells
    de = rng.normal(size=(spec.levels, S, 2)).astype(np.float32)
    _, _, corners = ofield.encode_fwd(spec, np.zeros(nt), xn)
    de_sf = de.transpose(1, 0, 2).reshape(S, 2 * spec.levels).astype(np.float64)
    gt, gtm = ofield.encode_bwd(spec, corners, de_sf, np.abs(de_sf), nt)
    X, DE = _t(torch, gpu, xn), _t(torch, gpu, de)
    for prec, tol in ((nsl.PRECISION_FP32, 1e-5), (nsl.PRECISION_MIXED, 2e-2)):
        for overwrite, before in ((True, 0.0), (False, 0.5)):
            G = torch.full((f.layout["total"],), 0.5, device=gpu)
            nsl.encode_bwd(f, X, DE, G, precision=prec, overwrite=overwrite)
            g = G.cpu().numpy().astype(np.float64)
            check_mag(f"single-bin scatter p{prec}", g[:nt], gt + before, gtm + before, tol)
            assert np.all(g[nt:] == 0.5)
            assert np.all(g[:nt][gtm == 0] == before)
