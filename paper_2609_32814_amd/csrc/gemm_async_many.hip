// The kernels of gemm_async.hip for many row types (star and graph laws, more
// than 16): a tile's class and column group are found by one bound a lane and
// a ballot.  The walk along up to 64 prefix entries, twice a tile, took a
// 64-type tile of one K step about 10 us (star law, activation gradient, q =
// 64, 16384 rows, 512 <- 3072: 308 -> 119 us; q = 32, 8407 rows, 2304 <- 512:
// 76 -> 38).  For few types the walk stays, in a build of its own: any other
// lookup in the same kernel gave it other registers and cost few-type
// products 1 to 5 % (a ballot: dense, q = 4, activation gradient of 512 rows,
// 768 <- 3072, 41.1 -> 43.1 us; halving: star, q = 3, forward of 4096 rows,
// 768 -> 3072, 28.2 -> 29.0 us, tensor law, weight gradient, 768 x 1536, 61.6
// -> 63.7).
#define STARQ_MANY_TYPES
#define star_gemm_async_kernel star_gemm_async_many_kernel
#include "gemm_async.hip"
