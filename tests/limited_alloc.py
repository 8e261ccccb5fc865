"""A workspace allocator (rcb_params.alloc / free) with a budget, for tests: it
refuses a block that would bring the bytes in use past `budget`, and one whose
size is in `sizes`."""


class LimitedAlloc:
    def __init__(self):
        import torch
        from paper_1108_0028_amd import _lib
        self.budget = 1 << 62
        self.sizes = set()
        self.live = self.peak = self.refused = 0
        self.blocks = {}

        def alloc(nbytes, stream, ctx):
            if nbytes in self.sizes or self.live + nbytes > self.budget:
                self.refused += 1
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(), stream or 0)
            self.blocks[p] = nbytes
            self.live += nbytes
            self.peak = max(self.peak, self.live)
            return p

        def free(ptr, stream, ctx):
            self.live -= self.blocks.pop(ptr)
            torch.cuda.caching_allocator_delete(ptr)

        self.alloc_fn = _lib._ALLOC_FN(alloc)
        self.free_fn = _lib._FREE_FN(free)

    def tree(self, monkeypatch, arrs, **options):
        """a Tree whose workspace comes from this allocator"""
        from paper_1108_0028_amd import Tree, _lib
        with monkeypatch.context() as mp:
            mp.setattr(_lib, "_TORCH_ALLOC", self.alloc_fn)
            mp.setattr(_lib, "_TORCH_FREE", self.free_fn)
            return Tree(*arrs, allocator="torch", **options)
