// Where the loads of a 16-row tile (csrc/gemm_common.h, FragRows, unchanged) go: a buffer load returns the address that it
// would read, or zeros past its descriptor's end.  No memory is touched, so tiles of any size can be asked for.  And which
// products have such tiles (csrc/gemm_decode.hip, choose_tile).
#include <stdio.h>
#include <string.h>

#include "gemm_decode.hip"

FiberIdx::operator unsigned() const { return 0; }
FiberIdx3 threadIdx;
dim3 blockIdx, blockDim, gridDim;
void __syncthreads() {}
uint32_t exchange(uint32_t, int) { return 0; }

namespace aed {  // not reached here
hipError_t launch_gemm_tiled(GemmEpi, const GemmArgs&, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_gemm_dma_crosskv(const GemmArgs&, hipStream_t) { return hipErrorInvalidValue; }
}  // namespace aed
using namespace aed;

// k blocks of a tile of K elements a row: the first, the last, and those around the offsets that 30, 31 and 32 bits hold
template <typename T> int check(long long K) {
    constexpr int ES = sizeof(T);
    char* const tile = reinterpret_cast<char*>(1ull << 44);
    int bad = 0;
    const long long last = K / 64 - 1;
    for (long long kb : {0ll, 1ll, (1ll << 30) / (1024 * ES) - 1, (1ll << 30) / (1024 * ES), (1ll << 31) / (1024 * ES), (1ll << 32) / (1024 * ES), last}) {
        if (kb > last) continue;
        for (int rows : {1, 7, 16})
            for (int lane = 0; lane < 64; ++lane) {
                Frag16<T> f;
                FragRows<ES>(tile, rows, lane).load((int)kb, f);
                uint64_t got[ES][2];
                static_assert(sizeof f == sizeof got, "a lane's 16 elements are ES pieces of 16 bytes");
                memcpy(got, &f, sizeof got);
                for (int j = 0; j < ES; ++j) {
                    const uint64_t want = (lane & 15) < rows
                        ? (uint64_t)(tile + frag_elem_off<ES>(lane & 15, (int)(kb * 64 + (lane >> 4) * 16 + j * 16 / ES), (int)K)) : 0;
                    if (got[j][0] != want && bad++ < 4)
                        printf("%d bytes an element, K %lld, block %lld, lane %d of %d rows, piece %d: %llx, not %llx\n", ES, K, kb, lane,
                               rows, j, (unsigned long long)got[j][0], (unsigned long long)want);
                }
            }
    }
    return bad;
}

template <typename T> int check_choice() {
    constexpr int kMaxK = FragRows<sizeof(T)>::kMaxK;
    int bad = 0, small = 0;
    for (int M : {1, 7, 16, 17, 48, 64, 100, 300})
        for (int N : {256, 512, 768, 1024, 2048})
            for (long long K : {256ll, 1024ll, 4096ll, 4352ll, (long long)kMaxK, kMaxK + 256ll, 2ll * kMaxK, 4ll * kMaxK}) {
                GemmArgs a = {};
                a.M = M; a.N = N; a.K = (int)K;
                const bool t11 = choose_tile<T, PRO_T>(a, N) == T11;
                small += t11;
                if (t11 && K > kMaxK && bad++ < 4) printf("%d bytes an element, %d x %d over %lld on 16-row tiles\n", (int)sizeof(T), M, N, K);
            }
    return bad + (small == 0);
}

int main() {
    int bad = check_choice<bf16_t>() + check_choice<float>();
    for (long long K : {256ll, 1024ll, 4096ll, 4352ll, 1ll << 24}) bad += check<bf16_t>(K) + check<float>(K);
    bad += check<bf16_t>(FragRows<2>::kMaxK);
    printf("%d wrong\n", bad);
    return bad != 0;
}
