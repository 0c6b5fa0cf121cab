// Group form of the CRT halves of the 6144-bit size class.
#define PMK_CLASS_BITS 6144
#include "kgroup.inc"
