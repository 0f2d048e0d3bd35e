"""Problems that the tile choice sends to the 256 x 256 kernels: checked by
test_launch_routes.py on the CPU, run by test_gpu_gemm_large.py.

FP4 and MXFP8: ragged edges; K of 1, 3 and 5 units of 128 (fewer than the LDS ring's
stages and more, with several tiles a workgroup, so that one tile's loads run into the
next one's) as well as long ones."""
SHORT_K = [(16400, 16390, 70), (8200, 16400, 384), (8200, 12301, 600)]
FP4 = [(2100, 4000, 1500), (3000, 4001, 1700), (4096, 4096, 2048)]
# K of whole 512 once padded to 128 (16-byte scale loads) and not
MXFP8 = [(2100, 4000, 700), (3000, 4001, 1100), (2100, 4000, 1024), (3000, 4001, 1536)]
MXFP8_ONE_PRODUCT = (16400, 16400, 64)
QUANTIZED = (4090, 4088, 4100)
# rows of the experts, N, K
GROUPED = [((0, 1500, 1, 2300, 255, 257, 0, 3700), 4000, 384), ((700,) * 16, 2720, 640)]
