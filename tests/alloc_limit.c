/* Device allocations counted, and refused above a limit, and those of pinned
   memory counted: loaded globally before a copy of the library, whose hipMalloc,
   hipFree and hipHostMalloc then are these. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <link.h>
#include <pthread.h>
#include <stddef.h>
#include <string.h>

enum { N = 1 << 16, OUT_OF_MEMORY = 2 };
static struct { void* p; size_t n; } held[N];
static size_t live, limit = (size_t)-1;
static pthread_mutex_t lock = PTHREAD_MUTEX_INITIALIZER;

static int find(struct dl_phdr_info* i, size_t size, void* out)
{
    (void)size;
    if (!strstr(i->dlpi_name, "libamdhip64.so")) return 0;
    *(void**)out = dlopen(i->dlpi_name, RTLD_LAZY | RTLD_NOLOAD);
    return *(void**)out != NULL;
}

static void* real(const char* name)
{
    void* h = NULL;
    dl_iterate_phdr(find, &h);
    return h ? dlsym(h, name) : NULL;
}

int hipMalloc(void** p, size_t n)
{
    static int (*f)(void**, size_t);
    if (!f) f = (int (*)(void**, size_t))real("hipMalloc");
    pthread_mutex_lock(&lock);
    int st = OUT_OF_MEMORY, i = 0;
    while (i < N && held[i].p) ++i;
    if (i < N && live + n <= limit && live + n >= live && (st = f(p, n)) == 0) {
        held[i].p = *p;
        held[i].n = n;
        live += n;
    }
    pthread_mutex_unlock(&lock);
    return st;
}

int hipFree(void* p)
{
    static int (*f)(void*);
    if (!f) f = (int (*)(void*))real("hipFree");
    pthread_mutex_lock(&lock);
    for (int i = 0; p && i < N; ++i)
        if (held[i].p == p) {
            live -= held[i].n;
            held[i].p = NULL;
            break;
        }
    pthread_mutex_unlock(&lock);
    return f(p);
}

static long pinned;
static int refuse_pinned;

int hipHostMalloc(void** p, size_t n, unsigned flags)
{
    static int (*f)(void**, size_t, unsigned);
    if (!f) f = (int (*)(void**, size_t, unsigned))real("hipHostMalloc");
    __atomic_add_fetch(&pinned, 1, __ATOMIC_RELAXED);
    return refuse_pinned ? OUT_OF_MEMORY : f(p, n, flags);
}

long pinned_calls(void) { return __atomic_load_n(&pinned, __ATOMIC_RELAXED); }
size_t alloc_live(void) { return live; }
void alloc_limit(size_t n) { limit = n; }
void pinned_refuse(int on) { refuse_pinned = on; }
