"""The many-row kernel's tile forms: the decoders of the device test reach each of them (on the 256
compute units of an MI355X) where the columns do not fill the last tile and K ranges differ in length."""
from tests import ring_forms


def test_workloads_reach_every_form_at_its_remainders():
    seen = ring_forms.covered()
    reached = {(kind, f) for _, kind, f, _, _ in seen}
    assert {f for _, f in reached} == set(range(len(ring_forms.forms())))
    partial = {(kind, f) for _, kind, f, rem, _ in seen if rem}
    for f, (mi, nj, *_) in enumerate(ring_forms.forms()):
        if nj > 2:  # (layer widths are multiples of 64: tiles of 64 columns are always whole)
            assert {("qkv", f), ("argmax", f), ("resid", f)} <= partial, f
            assert any(kind == "resid" and g == f and ranges == "uneven" for _, kind, g, _, ranges in seen), f
        if nj > 4:  # gate and up columns alternate in a tile: half as many features as columns
            assert ("gated", f) in partial, f
        assert ("argmax", f) in partial, f  # a vocabulary has any width
    assert {"store", "cross", "bias-gelu", "bias-resid"} <= {kind for kind, _ in reached}
