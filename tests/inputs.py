"""Test inputs whose recipe includes a statistic of the method: the encoder-FFN configuration's
per-token activation scales are the value training starts them from, 2 * mean|A| per token.  The
seeded generators hold no method arithmetic, so the tests derive the scales with the oracle and
hand the same values to both sides."""
import numpy as np

import oracle
import synth


def config2(which, M=4096):
    c = synth.config2(which, M=M)
    c["s_a"] = oracle.act_scale(c["A"])
    return c


def poison_gap(A, K):
    """Fill what lies between the ends of the rows (columns K on) with values that show wherever they are read: the
    largest magnitudes, of both signs and never of equal sum, with NaN among them for paths that must not fault on it."""
    A[:, K:] = np.resize(np.array([65504.0, -65504.0, 65504.0, np.nan, 65504.0], A.dtype), A.shape[1] - K)
