"""The C struct that a configuration keeps: it shows nowhere but in the calls, and a changed copy has its own."""
import copy
import dataclasses
import pickle

import paper_2312_17241_amd as cngp


def test_a_configuration_that_was_passed_is_still_a_value():
    make = lambda **over: cngp.Config(**{**dict(d=3, L=16, F=2, N_f=2**16, N_c=2**14, N_p=16, N_min=16, N_max=2048), **over})
    used, fresh = make(), make()
    assert used._ref()._obj.N_f == 2**16 and used._ref() is used._ref()
    assert used == fresh and hash(used) == hash(fresh) and repr(used) == repr(fresh) and used.__dict__ == fresh.__dict__
    for other in (pickle.loads(pickle.dumps(used)), copy.copy(used), copy.deepcopy(used), dataclasses.replace(used), cngp.Config(**used.__dict__)):
        assert other == used and other._ref() is not used._ref()
    assert dataclasses.replace(used, L=4)._ref()._obj.L == 4 and used._ref()._obj.L == 16
    m = cngp.MlpConfig(32, 3)
    assert m.weight_count == 64 * (32 + 64 + 3) and pickle.loads(pickle.dumps(m)) == m
