/* hipMalloc / hipFree with a cap on the bytes outstanding, for
 * tests/test_gpu_load_memory.py: loaded with global visibility before the
 * library, so that the library's calls come here first. */
#include <dlfcn.h>
#include <pthread.h>
#include <stddef.h>

enum { SLOTS = 4096, OUT_OF_MEMORY = 2 };
static struct {
    void *p;
    size_t n;
} blk[SLOTS];
static size_t held, peak, cap = (size_t)-1;
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static int (*real_malloc)(void **, size_t);
static int (*real_free)(void *);

int cap_init(const char *hip) {
    void *h = dlopen(hip, RTLD_NOW | RTLD_NOLOAD);
    if (!h) h = dlopen(hip, RTLD_NOW);
    if (!h) return 1;
    real_malloc = (int (*)(void **, size_t))dlsym(h, "hipMalloc");
    real_free = (int (*)(void *))dlsym(h, "hipFree");
    return real_malloc && real_free ? 0 : 2;
}
void cap_set(size_t bytes) { cap = bytes; }
size_t cap_held(void) { return held; }
size_t cap_peak(void) { return peak; }
void cap_reset_peak(void) { peak = held; }

int hipMalloc(void **p, size_t n) {
    pthread_mutex_lock(&mu);
    int rc = OUT_OF_MEMORY;
    *p = NULL;
    if (held + n <= cap && (rc = real_malloc(p, n)) == 0) {
        int i = 0;
        while (i < SLOTS && blk[i].p) ++i;
        if (i < SLOTS) {
            blk[i].p = *p;
            blk[i].n = n;
            held += n;
            if (held > peak) peak = held;
        }
    }
    pthread_mutex_unlock(&mu);
    return rc;
}
int hipFree(void *p) {
    pthread_mutex_lock(&mu);
    for (int i = 0; p && i < SLOTS; ++i)
        if (blk[i].p == p) {
            held -= blk[i].n;
            blk[i].p = NULL;
            break;
        }
    const int rc = real_free(p);
    pthread_mutex_unlock(&mu);
    return rc;
}
