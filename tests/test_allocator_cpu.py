"""The torch allocator's hooks are made once: objects release their memory through the hook that was
current when they were made, so setting it again must not free the callbacks they hold."""
from paper_1506_07577_amd import ebbx


def test_setting_the_torch_allocator_again_keeps_its_hooks():
    ebbx.lib()
    hooks = list(ebbx._hooks)
    assert len(hooks) == 2
    ebbx.use_torch_allocator(False)
    ebbx.use_torch_allocator(True)
    assert all(a is b for a, b in zip(ebbx._hooks, hooks))
