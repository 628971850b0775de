/* Counts the device memory that a library in the process allocates and the
 * graphs that it instantiates: loaded with RTLD_GLOBAL before that library, its
 * hipMalloc, hipFree and hipGraphInstantiate are these. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <pthread.h>
#include <stddef.h>

#define SLOTS 65536
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static struct { void *p; size_t n; } slot[SLOTS];
static size_t used, most;
static int (*real_malloc)(void **, size_t);
static int (*real_free)(void *);
static int (*real_instantiate)(void **, void *, void **, char *, size_t);
static int graphs, mallocs;

int count_init(const char *runtime)
{
    void *h = dlopen(runtime, RTLD_NOW);
    if (!h)
        return 1;
    *(void **)&real_malloc = dlsym(h, "hipMalloc");
    *(void **)&real_free = dlsym(h, "hipFree");
    *(void **)&real_instantiate = dlsym(h, "hipGraphInstantiate");
    return real_malloc && real_free && real_instantiate ? 0 : 2;
}

int hipMalloc(void **p, size_t n)
{
    const int rc = real_malloc(p, n);
    if (rc == 0 && *p) {
        pthread_mutex_lock(&mu);
        size_t k = ((size_t)*p >> 8) % SLOTS;
        while (slot[k].p)
            k = (k + 1) % SLOTS;
        slot[k].p = *p;
        slot[k].n = n;
        used += n;
        ++mallocs;
        if (used > most)
            most = used;
        pthread_mutex_unlock(&mu);
    }
    return rc;
}

int hipFree(void *p)
{
    if (p) {
        pthread_mutex_lock(&mu);
        for (size_t k = 0; k < SLOTS; ++k) /* (a slot is found by search: no order to keep) */
            if (slot[k].p == p) {
                used -= slot[k].n;
                slot[k].p = NULL;
                break;
            }
        pthread_mutex_unlock(&mu);
    }
    return real_free(p);
}

int hipGraphInstantiate(void **exec, void *graph, void **node, char *log, size_t n)
{
    __atomic_add_fetch(&graphs, 1, __ATOMIC_RELAXED);
    return real_instantiate(exec, graph, node, log, n);
}

int count_graphs(void) { return __atomic_load_n(&graphs, __ATOMIC_RELAXED); }
int count_mallocs(void) { return mallocs; }
size_t count_used(void) { return used; }
size_t count_most(void) { return most; }
void count_reset(void) { most = used; }
