// Error reporting and a device-wide exclusive scan shared by the library's
// entry points.
#include "bop_internal.h"

#include <cstring>
#include <mutex>
#include <vector>

namespace bop {

static thread_local char g_err[512];

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
}

// a device attribute of the current device, cached per (device, slot)
static int cached_attr(int slot, hipDeviceAttribute_t attr, int fallback)
{
    static std::mutex mu;
    static std::vector<int> cache[2];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fallback;
    std::lock_guard<std::mutex> lk(mu);
    std::vector<int> &c = cache[slot];
    if ((int)c.size() <= dev) c.resize(dev + 1, 0);
    if (!c[dev]) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, attr, dev) != hipSuccess || v <= 0) v = fallback;
        c[dev] = v;
    }
    return c[dev];
}

int device_cus() { return cached_attr(0, hipDeviceAttributeMultiprocessorCount, 256); }

int device_lds_per_block() { return cached_attr(1, hipDeviceAttributeMaxSharedMemoryPerBlock, 65536); }

// ---------------------------------------------------------------------------
// exclusive scan: up to SCAN_ONE items by one block in one launch (a launch costs more
// than the scan of so few); else 4096 items per block, the block totals scanned
// recursively, then added back.
// ---------------------------------------------------------------------------
constexpr int SCAN_T = 1024, SCAN_I = 4, SCAN_CHUNK = SCAN_T * SCAN_I;
constexpr long SCAN_ONE = 8 * SCAN_CHUNK;

// Exclusive prefix of v over the block, plus carry; total: the sum over the block.
__device__ inline int block_prefix(int v, int carry, int *s_w, int &total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        x += lane >= o ? y : 0;
    }
    __syncthreads();                  // the previous use of s_w is over
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    int below = 0;
    total = 0;
    for (int q = 0; q < SCAN_T / 64; ++q) {
        below += q < w ? s_w[q] : 0;
        total += s_w[q];
    }
    return carry + below + x - v;
}

// One chunk per block; with sums == NULL one block takes all chunks in turn and writes
// the total out[n].
__global__ void __launch_bounds__(SCAN_T)
scan_chunks(const int *__restrict__ in, int *__restrict__ out, long n, int *__restrict__ sums)
{
    __shared__ int s_w[SCAN_T / 64];
    int carry = 0;
    for (long c = (long)blockIdx.x * SCAN_CHUNK; c < n; c += SCAN_CHUNK) {
        const long base = c + (long)threadIdx.x * SCAN_I;
        int v[SCAN_I], t = 0, total;
        for (int k = 0; k < SCAN_I; ++k) {
            v[k] = (base + k < n) ? in[base + k] : 0;
            t += v[k];
        }
        int run = block_prefix(t, carry, s_w, total);
        for (int k = 0; k < SCAN_I; ++k) {
            if (base + k < n) out[base + k] = run;
            run += v[k];
        }
        carry += total;
        if (sums) break;
    }
    if (threadIdx.x == 0) {
        if (sums) sums[blockIdx.x] = carry;
        else out[n] = carry;
    }
}

// adds the chunks' offsets; the last block writes the total out[n]
__global__ void __launch_bounds__(SCAN_T)
scan_add(int *__restrict__ out, long n, const int *__restrict__ offs)
{
    long base = (long)blockIdx.x * SCAN_CHUNK + (long)threadIdx.x * SCAN_I;
    int o = offs[blockIdx.x];
    for (int k = 0; k < SCAN_I; ++k)
        if (base + k < n) out[base + k] += o;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = offs[gridDim.x];
}

size_t scan_scratch_bytes(long n)
{
    size_t b = 0;
    while (n > SCAN_ONE) {
        long nb = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
        b += align_up(sizeof(int) * (size_t)(2 * nb + 1), 256);
        n = nb;
    }
    return b + 256;
}

int exclusive_scan(const int *in, int *out, long n, void *scratch, hipStream_t stream)
{
    if (n <= SCAN_ONE) {
        scan_chunks<<<1, SCAN_T, 0, stream>>>(in, out, n < 0 ? 0 : n, nullptr);
        BOP_LAUNCHED();
        return BOP_OK;
    }
    long nb = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    int *sums = (int *)scratch;
    int *offs = sums + nb;
    char *next = (char *)scratch + align_up(sizeof(int) * (size_t)(2 * nb + 1), 256);
    scan_chunks<<<(unsigned)nb, SCAN_T, 0, stream>>>(in, out, n, sums);
    BOP_LAUNCHED();
    int rc = exclusive_scan(sums, offs, nb, next, stream);
    if (rc) return rc;
    scan_add<<<(unsigned)nb, SCAN_T, 0, stream>>>(out, n, offs);
    BOP_LAUNCHED();
    return BOP_OK;
}

}  // namespace bop

extern "C" int bop_last_error(char *buf, size_t n)
{
    size_t len = strlen(bop::g_err);
    if (buf && n) {
        size_t c = len < n - 1 ? len : n - 1;
        memcpy(buf, bop::g_err, c);
        buf[c] = 0;
    }
    return (int)len;
}
