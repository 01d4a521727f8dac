"""DsfqLinear's kept workspace with several threads, on the CPU: every order in which two first calls can write its state."""
import itertools
import threading

import pytest
import torch

from paper_2509_21302_amd import binding as q
from paper_2509_21302_amd.module import DsfqLinear

STEPS = 3                                 # a call's allocation and its writes to the layer: as many turns as it takes, and one more


class Turns:
    """Two threads take turns in a given order; one that has nothing left to do gives its turns away."""

    def __init__(self, order):
        self.order, self.done, self.cond, self.local = list(order), set(), threading.Condition(), threading.local()

    def step(self):
        me = getattr(self.local, "name", None)
        if me is None:
            return
        with self.cond:
            def my_turn():
                while self.order and self.order[0] in self.done:
                    self.order.pop(0)
                return not self.order or self.order[0] == me
            assert self.cond.wait_for(my_turn, timeout=30)
            if self.order:
                self.order.pop(0)
            self.cond.notify_all()

    def run(self, name, work):
        self.local.name = name
        try:
            work()
        finally:
            with self.cond:
                self.done.add(name)
                self.cond.notify_all()


class Layer(DsfqLinear):
    """A layer without device tensors; what it keeps of its workspace takes a turn to write."""

    def __init__(self, turns):
        self.N, self.K, self.packed, self.Wf = 1024, 512, True, None
        self._ws = (-1, None)
        self.turns = turns

    def __setattr__(self, name, value):
        if name.startswith("_ws") and hasattr(self, "turns"):
            self.turns.step()
        super().__setattr__(name, value)


@pytest.mark.parametrize("rows", [(1000, 10), (10, 1000)])
def test_two_first_calls_leave_a_workspace_that_fits(monkeypatch, rows):
    cpu = torch.device("cpu")
    for order in set(itertools.permutations([0] * STEPS + [1] * STEPS)):
        turns = Turns(order)
        layer = Layer(turns)
        empty = torch.empty

        def stepping_empty(*a, **kw):
            turns.step()
            return empty(*a, **kw)
        monkeypatch.setattr(torch, "empty", stepping_empty)
        got, errors = {}, []

        def call(i):
            try:
                turns.run(i, lambda: got.__setitem__(i, layer._workspace(rows[i], cpu)))
            except BaseException as e:
                errors.append(e)
        threads = [threading.Thread(target=call, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        monkeypatch.setattr(torch, "empty", empty)
        assert not errors, (order, errors)
        for i in range(2):
            assert got[i].numel() >= q.qvggt_workspace_bytes(rows[i], layer.N, layer.K), (order, "a call was given too little")
        for M in (1, 10, 11, 500, 1000, 1001):
            assert layer._workspace(M, cpu).numel() >= q.qvggt_workspace_bytes(M, layer.N, layer.K), (order, M)
