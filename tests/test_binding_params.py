"""The parameter block of the conveniences is the one that make_params gives, field by field."""
import pytest

from paper_2605_13473_amd import binding as ob


@pytest.mark.parametrize("hp", [ob.Hyper(), ob.Hyper(scale=0.25, eta=0.5, d_min=1, d_max=float("inf"), beta_aware=False),
                                ob.Hyper(segments=3, p1_pieces=-1, p1_piece_sweeps=2, p1_solved=1),
                                ob.Hyper(d_max=1e300),            # no finite float32
                                ob.Hyper(segments=2**31 + 5)])    # no int32
@pytest.mark.parametrize("bf16,ret_vec,gate_vec", [(False, False, True), (True, True, False)])
def test_packed_at_once(hp, bf16, ret_vec, gate_vec):
    args = (2, 3, 4, 128, 64, bf16, hp, ret_vec, gate_vec)
    assert bytes(ob._shape_params(*args)) == bytes(ob.make_params(*args))
