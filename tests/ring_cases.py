"""Forward products that reach every form of the tiles with direct loads (launch_recorder.RINGS), with and without stores past the caches: what test_gpu_ring_cases.py computes and
test_launches_host.py finds to take that form."""

# (M, N, K), form, stores past the caches (more than 64 M outputs in rows of whole lines).  The widest tiles over one to three K-tiles, fewer than their ring holds, several tiles to a block
MATRICES = [((124_079, 131, 256), "wide", False), ((131_072, 1500, 192), "wide", False), ((90_568, 768, 64), "wide", True), ((131_072, 1024, 128), "wide", True), ((70_001, 1056, 192), "wide", True),
            ((24_773, 777, 1024), "wide", False), ((124_393, 69, 384), "tall", False), ((234_168, 320, 256), "tall", True), ((16_482, 160, 64), "narrow", False), ((340_057, 288, 64), "narrow", True),
            ((38_503, 139, 64), "square", False), ((156_685, 576, 64), "square", True), ((4911, 198, 512), "low", False), ((64, 20_001, 128), "square", False), ((1, 40_000, 1024), "square", False)]

# (B, H, W, C, N, R, S, stride, pad), form, stores past the caches.  Whole K-tiles to a tap (C a multiple of 64), and K-tiles across taps
LAYERS = [((12, 36, 55, 128, 352, 2, 2, 1, 1), "wide", False), ((501, 6, 54, 64, 416, 1, 1, 1, 0), "wide", True), ((80, 50, 51, 112, 144, 3, 3, 2, 1), "wide", False),
          ((9, 65, 58, 64, 312, 3, 3, 1, 1), "tall", False), ((314, 64, 51, 128, 352, 1, 1, 2, 0), "tall", True), ((42, 17, 68, 160, 140, 2, 2, 1, 1), "tall", False), ((129, 34, 45, 176, 352, 1, 1, 1, 0), "tall", True),
          ((126, 30, 20, 256, 20, 2, 2, 1, 1), "narrow", False), ((464, 58, 10, 32, 32, 5, 5, 2, 2), "narrow", False), ((98, 26, 52, 16, 608, 1, 1, 1, 0), "narrow", True),
          ((129, 28, 4, 384, 288, 1, 1, 1, 0), "square", False), ((429, 19, 14, 16, 68, 3, 3, 1, 1), "square", False),
          ((2, 4, 10, 320, 32, 1, 1, 2, 0), "low", False), ((3, 4, 4, 32, 144, 1, 1, 2, 0), "low", False), ((2, 7, 7, 48, 132, 3, 3, 1, 1), "low", False), ((4, 5, 5, 512, 64, 3, 3, 1, 1), "low", False)]
