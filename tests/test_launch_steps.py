"""lbm_launch_steps without a handle (no GPU needed)."""


def test_launch_steps_refuses_a_null_handle():
    from paper_1701_00702_amd import lbm
    assert lbm.lbm_launch_steps(None)[0] == -1
    assert lbm._lib.lbm_launch_steps(None, None, None) == -1
    assert lbm.lbm_last_error()
    assert lbm._lib.lbm_reset_launch(None) == -1 and lbm.lbm_last_error()
